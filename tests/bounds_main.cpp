/*
 * Test driver: the arithmetic of csrc/bounds.h, deal.h and errors.h on the host, built by
 * tests/test_bounds_cpu.py with the undefined-behaviour sanitizer.  CPU-only
 * test infrastructure.
 *
 * "counts": stdin n_rows_max, E_loc, E_loc counts; stdout the rows that each
 * group keeps and whether any count was changed.  The lanes of a wave take the
 * steps of the device's scan one after the other.
 */
#include <cstdio>
#include <cstring>

#include "bounds.h"
#include "deal.h"
#include "errors.h"

using namespace moe;

static int counts()
{
    int cap, n;
    if (std::scanf("%d %d", &cap, &n) != 2 || n < 0 || n > 256) return 2;
    int32_t carry = 0;
    bool bad = false;
    for (int c0 = 0; c0 < n; c0 += 64) {
        int32_t c[64] = {}, asked[64], x[64], y[64];
        for (int l = 0; l < 64; ++l) {
            if (c0 + l < n && std::scanf("%d", &c[l]) != 1) return 2;
            x[l] = asked[l] = rows_asked(c[l], cap);
        }
        for (int o = 1; o < 64; o <<= 1) {
            std::memcpy(y, x, sizeof x);
            for (int l = o; l < 64; ++l) x[l] = add_capped(x[l], y[l - o], cap);
        }
        for (int l = 0; l < 64 && c0 + l < n; ++l) {
            const int32_t keep = rows_kept(asked[l], add_capped(carry, l ? x[l - 1] : 0, cap), cap);
            bad |= keep != c[l];
            std::printf("%d ", keep);
        }
        carry = add_capped(carry, x[63], cap);
    }
    std::printf("%d\n", (int)bad);
    return 0;
}

/* "blocks": stdin n, then n pairs of blocks and columns; stdout per pair the
 * blocks that a tile may have, and whether such rows are taken at all. */
static int blocks()
{
    int n;
    if (std::scanf("%d", &n) != 1) return 2;
    for (; n > 0; --n) {
        int most;
        long long cols;
        if (std::scanf("%d %lld", &most, &cols) != 2) return 2;
        std::printf("%d %d ", tile_blocks(most, cols), (int)tile_fits(kLeastBlocks, cols));
    }
    std::printf("\n");
    return 0;
}

/* "status": stdin n, then n values of the error word; stdout their statuses. */
static int status()
{
    int n, err;
    if (std::scanf("%d", &n) != 1) return 2;
    for (; n > 0 && std::scanf("%d", &err) == 1; --n) std::printf("%d ", (int)sticky_status(err));
    std::printf("\n");
    return n;
}

/* "deal": stdin workgroups, gate/up items, down items, phases, bytes of a row;
 * stdout the fixed item of each workgroup, then for each product and list its length and items. */
static int deal()
{
    int P, g, d, phases, bytes;
    if (std::scanf("%d %d %d %d %d", &P, &g, &d, &phases, &bytes) != 5) return 2;
    Deal q;
    q.count(P, g, d, phases);
    q.deal(P, g, d, bytes);
    std::printf("%d %d ", 1 << q.lg, q.C);
    for (int b = 0; b < P; ++b) std::printf("%d ", q.fixed(b));
    for (int p = 0; p < 2; ++p)
        for (int y = 0; y < 1 << q.lg; ++y) {
            std::printf("%d ", q.len(p, y));
            for (int j = 0; j < q.len(p, y); ++j) std::printf("%d ", q.item(j, y, p));
        }
    std::printf("\n");
    return 0;
}

/* "split": stdin n, then n times streams, fp8, items, bytes of weights,
 * workgroups; stdout whether the products are launched one by one. */
static int split()
{
    int n;
    if (std::scanf("%d", &n) != 1) return 2;
    for (; n > 0; --n) {
        int streams, fp8, grid;
        long long items, bytes;
        if (std::scanf("%d %d %lld %lld %d", &streams, &fp8, &items, &bytes, &grid) != 5) return 2;
        std::printf("%d ", (int)split_products(streams, fp8 != 0, items, bytes, grid));
    }
    std::printf("\n");
    return 0;
}

int main(int argc, char **argv)
{
    if (argc < 2) return 2;
    if (!std::strcmp(argv[1], "counts")) return counts();
    if (!std::strcmp(argv[1], "blocks")) return blocks();
    if (!std::strcmp(argv[1], "status")) return status();
    if (!std::strcmp(argv[1], "deal")) return deal();
    if (!std::strcmp(argv[1], "split")) return split();
    return 2;
}
