// How the items of an FFN pass are dealt to the work lists of ffn_sched.h: plain
// constexpr arithmetic without HIP types, checked on the host.
#pragma once

#include <stdint.h>

namespace moe {

constexpr int kListsLog2 = 3;
constexpr int kLists = 1 << kListsLog2;

// Rows shorter than this (bytes) are short, see deal().
constexpr int kShortRow = 1024;

// Product p (0 gate/up, 1 down) deals its items in runs of consecutive ones to
// the lists in turn.  Workgroup b belongs to list b % lists.
struct Deal {
    int lg = 0;                // log2 of the lists
    int C = 1, C1 = 1;         // run lengths of the gate/up and of the down items
    int total0 = 0, total1 = 0;

    // P workgroups; g gate/up and d down items, of which the launch runs those
    // of `phases` (1, 2, or 3 for both); row_bytes: of an activation row.
    constexpr void deal(int P, int g, int d, int phases, int64_t row_bytes)
    {
        lg = (P & (kLists - 1)) ? 0 : kListsLog2;
        total0 = (phases & 1) ? g : 0;
        total1 = (phases & 2) ? d : 0;
        // One item for each of a list's workgroups.  Fewer items than
        // workgroups are shared evenly: in runs of P / lists they fill the first
        // lists only, and their weights come through those XCDs (32 items of one
        // expert, d = 7168, f = 2048, 16 rows, a layer: 79.0 us, shared 69.8; fp8,
        // two experts 80.4 and 58.8).  Not where rows are so short that the
        // weights do not count: latencies are lower with h in one L2 then (4
        // experts, f = d / 2, 64 tokens, shared and in runs: fp8, d = 512 31.8 and
        // 30.8, bf16, d = 256 25.5 and 24.2; bf16, d = 512, rows of 1 KB, 27.6 and
        // 28.1).
        const int share = (g + (1 << lg) - 1) >> lg, most = P >> lg;
        C = row_bytes < kShortRow ? most : share < 1 ? 1 : share < most ? share : most;
        // A list's down items are those of the row tiles that it did the
        // gate/up items of (as far as runs of one length allow): they are ready
        // when its own gate/up items are.
        const int c1 = (int)((float)C * (float)d / (float)(g > 1 ? g : 1) + 0.5f);
        C1 = c1 > 1 ? c1 : 1;
    }
    // Length of list y, and its j-th item.
    constexpr int len(int p, int y) const
    {
        const int R = p ? C1 : C, total = p ? total1 : total0;
        const int full = total / (R << lg), rem = total - full * (R << lg) - y * R;
        return full * R + (rem < 0 ? 0 : rem < R ? rem : R);
    }
    constexpr int item(int j, int y, int p) const
    {
        const int R = p ? C1 : C, r = j / R;
        return r * (R << lg) + y * R + (j - r * R);
    }
    // The fixed first item of workgroup b, or -1: the first C of each list's
    // gate/up items are fixed.
    constexpr int fixed(int b) const
    {
        const int j = b >> lg, it = (b & ((1 << lg) - 1)) * C + j;
        return j < C && it < total0 ? it : -1;
    }
};

}  // namespace moe
