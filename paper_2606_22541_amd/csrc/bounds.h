// Bounds on rows and tiles: plain constexpr arithmetic without HIP types, used
// by kernels and host code alike and checked on the host.
#pragma once

#include <stdint.h>

namespace moe {

// a + b, or `cap` where the sum is more (0 <= a, b <= cap): a running total of
// capped values never wraps, and capping the parts caps the whole alike.
constexpr int32_t add_capped(int32_t a, int32_t b, int32_t cap)
{
    return (uint32_t)a + (uint32_t)b < (uint32_t)cap ? a + b : cap;
}

// Pre-grouped counts: rows that a group of `count` rows (any value) can ask
// for in a buffer of `cap` rows, and those it keeps after `before` rows
// (0 <= before <= cap) of the groups ahead of it.
constexpr int32_t rows_asked(int32_t count, int32_t cap) { return count < 0 ? 0 : count < cap ? count : cap; }
constexpr int32_t rows_kept(int32_t asked, int32_t before, int32_t cap)
{
    return asked < cap - before ? asked : cap - before;
}

// A tile addresses its rows of activations and of outputs, `cols` elements
// each, with 32-bit byte offsets: the 32-row blocks that a bf16 tile of up to
// `most` may have, and whether the kernels take rows of that length at all
// (in tiles of kLeastBlocks blocks).
constexpr int kLeastBlocks = 8;
constexpr bool tile_fits(int blocks, int64_t cols) { return 32 * blocks * cols * 2 < (int64_t)1 << 31; }
constexpr int tile_blocks(int most, int64_t cols)
{
    while (most > kLeastBlocks && !tile_fits(most, cols)) --most;
    return most;
}

}  // namespace moe
