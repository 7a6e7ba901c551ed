// How the items of an FFN pass are dealt to the work lists of ffn_sched.h, and
// whether one launch runs both products: plain constexpr arithmetic without HIP
// types, checked on the host.
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
    // of `phases` (1, 2, or 3 for both).
    constexpr void count(int P, int g, int d, int phases)
    {
        lg = (P & (kLists - 1)) ? 0 : kListsLog2;
        total0 = (phases & 1) ? g : 0;
        total1 = (phases & 2) ? d : 0;
    }
    // The run lengths, after count(); row_bytes: of an activation row.
    constexpr void deal(int P, int g, int d, int64_t row_bytes)
    {
        // One item for each of a list's workgroups.  Up to three quarters as
        // many items as workgroups are shared evenly: in runs of P / lists they
        // fill the first lists only, and their weights come through those XCDs
        // (32 items of one expert, d = 7168, f = 2048, 16 rows, a layer: 79.0 us,
        // shared 69.8; fp8, two experts 80.4 and 58.8).  With more the lists are
        // nearly full, and runs that begin where a group does share its rows and
        // panels in one L2 (fp8, d = 7168, f = 2048, 192 items 114.5 and shared 112.4, 208
        // 112.8 and 113.3, 240 112.5 and 115.3; bf16, 100 rows an expert, 192 items
        // 123.7 and 123.1, 224 130.2 and 133.5).  Nor where rows are so short that
        // the weights do not count: latencies are lower with h in one L2 then (4
        // experts, f = d / 2, 64 tokens, shared and in runs: fp8, d = 512 31.8 and
        // 30.8, bf16, d = 256 25.5 and 24.2; bf16, d = 512, rows of 1 KB, 27.6 and
        // 28.1).
        const int share = (g + (1 << lg) - 1) >> lg, most = P >> lg;
        C = row_bytes < kShortRow || 4 * share > 3 * most ? most : share > 1 ? share : 1;
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

// A pass whose weights take at least about 30 us to stream, see split_products().
constexpr int64_t kLongStream = (int64_t)160 << 20;

// Whether a pass runs its products in a launch each, when the stage's passes
// come in on `streams` streams.  groups: its experts; rows: rows that one of them
// can expect, of tiles of up to `tile` rows and `nt` column tiles in the gate/up
// product; weight_bytes: of all its experts; grid: workgroups of a launch.
//
// One launch runs both faster when it has the GPU to itself, but its workgroups
// keep their CUs from the first item to the last, those that wait for the down
// product's rows included.  If the gate/up product is one round at most they wait
// most, and passes of other streams could have run there (us a micro-batch, d =
// 7168, f = 2048, 8 of 256 experts, top 8, one launch and two): bf16 on three
// streams T = 1024 125.3 and 119.0, T = 8192 262.6 and 242.3, on four T = 4096 181.5 and
// 161.5; fp8 on two streams T = 1024 89.6 and 69.3, on three T = 4096 103.6 and 95.5.
// Not otherwise:
//  * of several rounds, one launch fills the first product's last: fp8, two streams, T =
//    16384 283 and 320; 32 experts and a shared one, T = 1000, 495 and 511;
//  * bf16 on two streams: T = 4096 176 and 181, T = 1024 125.6 and 127.4;
//  * short passes are bound by their launches: 8 experts, top 2, three streams,
//    fp8, d = 2048, f = 1536 (75 MB) 22.7 and 24.0, bf16 (151 MB) 53.1 and 56.0, but
//    d = 4096, f = 1024 (201 MB) 56.0 and 44.1.
constexpr bool split_products(int streams, bool fp8, int64_t items, int64_t weight_bytes, int grid)
{
    return streams >= (fp8 ? 2 : 3) && weight_bytes >= kLongStream && items <= grid;
}

}  // namespace moe
