// Shared definitions of the gfx950 (CDNA4) kernels of the MoE expert stage.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bounds.h"
#include "errors.h"

namespace moe {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

// Dispatch: slots handled by one workgroup of the histogram / scatter kernels.
constexpr int kDispatchThreads = 256;
constexpr int kDispatchChunk = 1024;            // 4 slots per thread
constexpr int kMaxExperts = 1024;               // LDS histogram size
constexpr int kMaxLocalExperts = 256;
constexpr int kMaxLayers = 1024;
constexpr int kMaxIngestWords = 4096;            // ready words one ingest wait may poll
constexpr uint32_t kDefaultIngestSpins = 1u << 19;   // about a second of polling

// bf16 large tiles: 32-row blocks of each half of a tile.
constexpr int kHalfBlocks = 5;
constexpr int kTileBlocks = 2 * kHalfBlocks;
// Row tiles of a raster band: 4 x 320 rows of K = 7168 are read from L2 by the
// items of a band while their weight panels stream past; 2 and 8 measured the
// same within 0.5% (T = 32768), 1 reads every panel again per row tile.
constexpr int kBandBf16 = 4;
// fp8 tiles: up to 128 rows.
constexpr int kTileBlocksFp8 = 4;
constexpr int kBandFp8 = 8;

// Cache-policy operand of the raw buffer loads: non-temporal (streaming)
// data, read once, evicted first and kept out of the last-level cache.
constexpr int kNonTemporal = 2;

// Groups with at most this many rows ("small": an EP32 share at T = 4096 has
// ~128 rows per expert) take one tile of all their rows and 128 columns in the
// gate/up product, which streams each weight panel exactly once into
// registers; larger groups take large tiles (up to 320 rows, 256 columns).  The
// line is what a small tile's accumulators hold.  A pass with T k at most this
// has no large group in either product and runs the kernel without large
// tiles.
constexpr int kSmallRows = 192;
// The down product's line: groups of a few dozen rows (cold experts of skewed
// routing) stream their weights faster in small tiles.  Larger groups do not:
// with small down tiles up to 128 rows the pass at T = 4096 took 187 us instead
// of 180, up to 192 rows 213.
constexpr int kSmallRowsDown = 64;
static_assert(kSmallRows <= 32 * kLeastBlocks && kTileBlocksFp8 <= kLeastBlocks, "every tile's offsets fit");

__device__ __forceinline__ int lane_id() { return __lane_id(); }

// Round-to-nearest-even fp32 -> bf16 (finite inputs).
__device__ __forceinline__ bf16 f2bf(float v) { return static_cast<bf16>(v); }
__device__ __forceinline__ float bf2f(bf16 v) { return static_cast<float>(v); }

// Two fp32 values as a pair of bf16 in one word (round to nearest even), the
// first in the low half.
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    const bf16x2_t v = {static_cast<bf16>(lo), static_cast<bf16>(hi)};
    return __builtin_bit_cast(uint32_t, v);
}

// SiLU(g) * u = g / (1 + e^-g) * u with the hardware exp2 and reciprocal
// (about 1 ulp each in fp32, far below the bf16 rounding of the result).
// g -> -inf gives e = inf and a zero reciprocal; g -> +inf gives g * u.
__device__ __forceinline__ float silu_mul(float g, float u)
{
    const float e = __builtin_amdgcn_exp2f(-1.44269504088896341f * g);
    return g * __builtin_amdgcn_rcpf(1.0f + e) * u;
}

// Swaps lanes 32..63 of x with lanes 0..31 of y (v_permlane32_swap): after
// it, x holds [x.lo, y.lo] and y holds [x.hi, y.hi].
__device__ __forceinline__ void swap_halves(uint32_t &x, uint32_t &y)
{
    const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
    x = r[0];
    y = r[1];
}

// e4m3 (OCP E4M3FN) code of v, round to nearest even.  |v| is clamped to 448
// first, which makes the conversion saturating.
__device__ __forceinline__ uint32_t e4m3_pack4(float a, float b, float c, float d)
{
    a = fminf(fmaxf(a, -448.0f), 448.0f);
    b = fminf(fmaxf(b, -448.0f), 448.0f);
    c = fminf(fmaxf(c, -448.0f), 448.0f);
    d = fminf(fmaxf(d, -448.0f), 448.0f);
    int v = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, 0, false);
    v = __builtin_amdgcn_cvt_pk_fp8_f32(c, d, v, true);
    return (uint32_t)v;
}

}  // namespace moe
