// bf16 expert FFN (the MoE "GMM": hidden states on the left, one expert's
// weights on the right; section 3.4.2): both grouped products of a pass,
//
//   H[g] = SiLU(A[g] Wg[g]^T) * (A[g] Wu[g]^T),   Y[g] = H[g] Wd[g]^T,
//
// in one launch (or, where passes of several streams share the GPU, in one each:
// split_products()), for every group g (a local expert, or the shared expert).
// A[g] is a run of token rows (gathered from x through slot_of_row), all
// operands are K-contiguous, and the weights are stored in MFMA fragment
// order (see launch_pack_frag_bf16).
//
// One persistent workgroup of eight wave64s per CU takes work items (an
// output tile of one product) from device-built lists, so the host never
// learns the per-expert row counts and empty experts own no items.  Two kinds
// of tile share the launch:
//  * large (256 columns, up to 320 rows): bound by the matrix cores;
//  * small (128 columns, all of a group's up to 192 rows): bound by the HBM
//    stream of the group's weights.
//
// Items and their order (ffn_sched.h).  The items of the gate/up product come
// before those of the down product, and a down item starts as soon as every
// gate/up tile of its rows is written, so neither product has an idle last
// round and no launch gap separates them.
//
// Measured, against one launch per product and size class with whole rounds of
// equal tiles (us a micro-batch with its dispatch and combine, d = 7168, f =
// 2048, 8 of 256 experts here, top 8): T = 32768 810 -> 705, T = 8191 340 -> 258,
// T = 4096, where the weights' stream bounds both products, 168 -> 167; 32
// experts here and a shared one, T = 1000: 701 -> 537.
#pragma once

#include "ffn_sched.h"
#include "kernels.h"

namespace moe {

namespace {

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kRowElems = 32;                 // a large tile's LDS token row: 64 bytes
constexpr int kHalfRows = 32 * kHalfBlocks;   // rows of a large tile's half
constexpr int kRowsElems = 2 * kHalfRows * kRowElems;
constexpr int kStageElems = kRowsElems + 8192;   // ... and 16 KB of weight fragments: 36 KB
typedef __attribute__((address_space(3))) void lds_void;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *base, int64_t bytes)
{
    // Raw buffer: loads whose vector offset is at or past num_records return 0,
    // stores there are dropped.
    int32_t n = bytes > 0x7fffffff ? 0x7fffffff : (int32_t)bytes;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, n, 0x00020000);
}

// The LDS ring of a workgroup: four stages of 36 KB (separate __shared__
// arrays, indexed by compile-time constants, which keeps the compiler from
// waiting for every direct-to-LDS load in flight before an LDS read).  Large
// tiles keep token rows in a(S) and weight fragments in b(S).
struct Lds {
    bf16 *s[4];
    __device__ __forceinline__ bf16 *a(int i) const { return s[i]; }
    __device__ __forceinline__ bf16 *b(int i) const { return s[i] + kRowsElems; }
};

// One output tile of either product.
struct Out {
    __amdgpu_buffer_rsrc_t r;   // the tile's output rows, whole rows of `ld` elements
    int ld;
    bool swiglu;                // gate/up: h = SiLU(gate) * up; else the product itself
};

// Output of one 32x32 block of the transposed product D[feature][token]
// (v_mfma_f32_32x32x16_bf16 with the weights as its row operand): lane l
// holds token l % 32, and register r holds feature 8 (r/4) + 4 (l/32) + r%4
// of the block.  Lanes l and l ^ 32 hold the same token, so after swapping
// halves each lane has 8 consecutive features, 16 bytes.
//
// y_block: the block's 32 features, to memory.  tok: the lane's tile row; rows
// past the tile's fall outside the buffer range and are dropped.
__device__ __forceinline__ void y_block(const f32x16 &v, const Out &o, int tok, int col, bool present)
{
    const int hi = (__lane_id() >> 5) * 8;
    uint32_t p[8];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        p[2 * q] = pack_bf16x2(v[4 * q], v[4 * q + 1]);
        p[2 * q + 1] = pack_bf16x2(v[4 * q + 2], v[4 * q + 3]);
    }
    swap_halves(p[0], p[2]);
    swap_halves(p[1], p[3]);
    swap_halves(p[4], p[6]);
    swap_halves(p[5], p[7]);
    const int off = present ? (tok * o.ld + col + hi) * 2 : (int)0x80000000u;
    __builtin_amdgcn_raw_buffer_store_b128((u32x4){p[0], p[1], p[2], p[3]}, o.r, off, 0, 0);
    __builtin_amdgcn_raw_buffer_store_b128((u32x4){p[4], p[5], p[6], p[7]}, o.r, off + 32, 0, 0);
}

// h_block: SwiGLU.  The packed gate/up weights interleave by 16, so register
// r (r < 8) and r + 8 of a lane are gate and up of one h column; lane l returns
// h columns 8 (l / 32) .. + 7 of the block's 16.
__device__ __forceinline__ u32x4 h_block(const f32x16 &v)
{
    uint32_t p[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
        p[q] = pack_bf16x2(silu_mul(v[2 * q], v[2 * q + 8]), silu_mul(v[2 * q + 1], v[2 * q + 9]));
    swap_halves(p[0], p[2]);
    swap_halves(p[1], p[3]);
    return (u32x4){p[0], p[1], p[2], p[3]};
}

// H goes past this XCD's L2 to memory (agent scope): the down items that read
// it run on other XCDs in the same launch, and an item is counted as written
// only when memory has taken its stores.  The rows are staged in LDS so that
// they leave as whole 128-byte lines: written 32 bytes at a time, with HBM
// busy, some tiles' stores took 10 us to be taken.
__device__ __forceinline__ void h_store(u32x4 v, const Out &o, int off)
{
    constexpr int kAgentScope = 16;     // sc1
    __builtin_amdgcn_raw_buffer_store_b128(v, o.r, off, 0, kAgentScope);
}

// ---------------------------------------------------------------------------
// Large tiles: up to 320 rows x 256 columns.
//
// Eight waves (two per SIMD), wave w owning columns 64 (w % 4) .. + 63 and one
// half of the tile's nb 32-row blocks (w / 4: the first ceil(nb / 2) blocks or
// the rest), as NMB x 2 blocks of v_mfma_f32_32x32x16_bf16.  Both operands are
// staged once per workgroup in LDS; K advances 32 per step through a 4-deep
// ring of 36 KB stages (up to 20 KB of token rows, 16 KB of weight fragments)
// filled by direct-to-LDS loads kAhead = 2 steps ahead, issued one at a time
// between the MFMAs (the per-CU load path takes a 1 KB load about every 19
// clocks, and a burst of every wave's loads stalled the waves behind it).
// The two waves of a SIMD (w and w + 4) run in opposite phases: in phase E of
// step j waves 0..3 read step j's operands from LDS while waves 4..7 run step
// j-1's MFMAs, and in phase O the roles swap; a workgroup barrier separates
// the phases.  The fills of step j+2 go into the stage of step j-2, which both
// halves have read by then; before the barrier that opens phase E of step j
// each wave waits for its own fills of step j.  Every step issues the same
// loads (steps past K re-read the last one), so that wait is a constant.
//
// Token rows are 64 bytes per step in LDS, their 16-byte chunks XOR-swizzled
// by (row / 4) % 4 so that the 16-lane groups of each ds_read_b128 hit 64
// distinct banks; weight fragments are contiguous in memory (one 16 KB run of
// the panel-ordered weights per step) and read back lane-contiguous.
// ---------------------------------------------------------------------------
constexpr int kBK = 32;                       // bf16 elements per K step (2 MFMA sub-steps)
// Steps that the fills run ahead.  Two, of a ring of four: three are 0.3 to 0.6%
// slower (T = 32768 704 against 701 us, T = 8191 the same), since a step lasts
// longer than its loads take to come back.
constexpr int kAhead = 2;

struct Tile {
    __amdgpu_buffer_rsrc_t ra, rb;
    int KT;
    int ncb;           // weight column blocks present in the tile (8, or fewer at N's end)
    int stepb;         // bytes of one K step of the tile's weight panel (ncb x 2 KB)
    int va[3];         // token fills: offsets of this lane's rows of row groups 0..2, swizzled chunk
};

struct WaveConst {
    int voff_b;        // weight fill: lane * 16
    int a_rd;          // LDS element offset of this lane's token row (block 0)
    int b_rd;          // LDS element offset of this lane's weight fragment (block 0)
    int a_wr[3];       // LDS element offsets of the wave's row groups
    int wave, rd_hi, swz;
};

// Token-row loads of a wave whose half holds NMB blocks: its half's 2 NMB
// groups of 16 rows are loaded by four waves.
constexpr int row_loads(int nmb) { return (nmb + 1) / 2; }

// Staging of a gate/up tile's h in the ring after the K loop: row block i
// (first half 0.., second kHalfBlocks..) of 32 rows x 128 columns, padded so
// that neither side conflicts, three blocks to a stage.
constexpr int kHStride = 128 + 8;
static_assert(3 * 32 * kHStride <= kStageElems && 4 * 3 >= kTileBlocks, "h fits the ring");
__device__ __forceinline__ bf16 *h_stage(const Lds &l, int i)
{
    return l.s[i / 3] + (i % 3) * 32 * kHStride;
}

// Fills of step j, row_loads(NMB) + 2 per wave:
//  * row groups of 16 rows x 64 bytes, lane l -> row l / 4 of the group,
//    physical chunk l % 4 <- global chunk (l % 4) ^ ((row / 4) % 4);
//  * weight fragments: the stage holds 8 column blocks x 2 sub-steps, 1 KB
//    each, in that order; wave w loads fragments 2 w and 2 w + 1.
// Steps past K re-read the last step.  The row offset is in the vector
// offset, which the buffer range check covers (rows past the tile read as
// zero); the scalar offset, which it does not cover, only moves along K and
// between weight column blocks that exist (absent ones re-read the last).
// STREAM: a group of one row tile reads each of its weight panels once in
// the launch, so those loads are non-temporal: the panels do not displace
// what the caches hold for later kernels (the combine's rows) and the dirty
// lines of earlier ones.  Groups of several row tiles share their panels
// through L2 and keep ordinary loads.
template <int NMB, bool STREAM>
__device__ __forceinline__ void fill_one(const Tile &t, const WaveConst &w, bf16 *sa, bf16 *sb, int j, int i)
{
    const int js = min(j, t.KT - 1);
    if (i < row_loads(NMB)) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(t.ra, (lds_void *)(sa + w.a_wr[i]), 16, t.va[i],
                                                 js * kBK * 2, 0, 0);
    } else {
        const int f = w.wave * 2 + (i - row_loads(NMB));       // fragment of the stage: 2 cb + kk
        const int cb = min(f >> 1, t.ncb - 1), kk = f & 1;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            t.rb, (lds_void *)(sb + f * 512), 16, w.voff_b,
            js * t.stepb + (cb * 2 + kk) * 1024, 0, STREAM ? kNonTemporal : 0);
    }
}

template <int NMB, bool STREAM>
__device__ __forceinline__ void fill(const Tile &t, const WaveConst &w, bf16 *sa, bf16 *sb, int j)
{
#pragma unroll
    for (int i = 0; i < row_loads(NMB) + 2; ++i) fill_one<NMB, STREAM>(t, w, sa, sb, j, i);
}

template <int S, int NMB>
__device__ __forceinline__ void read_step(const WaveConst &w, const Lds &l, bf16x8 (&a0)[kHalfBlocks],
                                          bf16x8 (&a1)[kHalfBlocks], bf16x8 (&b0)[2], bf16x8 (&b1)[2])
{
    if constexpr (NMB > 0) {
        const bf16 *As = l.a(S);
        const bf16 *Bs = l.b(S);
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const int ch = ((kk * 2 + w.rd_hi) ^ w.swz) << 3;
#pragma unroll
            for (int mb = 0; mb < NMB; ++mb)
                (kk ? a1 : a0)[mb] = *(const bf16x8 *)&As[w.a_rd + mb * 32 * kRowElems + ch];
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
                (kk ? b1 : b0)[nb] = *(const bf16x8 *)&Bs[w.b_rd + (nb * 2 + kk) * 512];
        }
    }
}

// The 4 NMB MFMAs of one step, with this wave's fills of step jf spread
// among them when FILL; a wave without row blocks only fills its weight
// fragments.
template <int NMB, bool STREAM, bool FILL>
__device__ __forceinline__ void mma_step(const Tile &t, const WaveConst &w, bf16 *sa, bf16 *sb, int jf,
                                         f32x16 (&acc)[NMB > 0 ? NMB : 1][2], const bf16x8 (&a0)[kHalfBlocks],
                                         const bf16x8 (&a1)[kHalfBlocks], const bf16x8 (&b0)[2],
                                         const bf16x8 (&b1)[2])
{
    if constexpr (NMB == 0) {
        if constexpr (FILL) fill<0, STREAM>(t, w, sa, sb, jf);
    } else {
        constexpr int kM = 4 * NMB, kFills = row_loads(NMB) + 2, kEvery = kM / kFills;
        int nf = 0;
#pragma unroll
        for (int q = 0; q < kM; ++q) {
            const int kk = q / (2 * NMB), r = q % (2 * NMB), mb = r >> 1, nb = r & 1;
            acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kk ? b1[nb] : b0[nb], kk ? a1[mb] : a0[mb],
                                                                 acc[mb][nb], 0, 0, 0);
            if (FILL && q % kEvery == kEvery / 2 && nf < kFills) {
                fill_one<NMB, STREAM>(t, w, sa, sb, jf, nf);
                ++nf;
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
}

__device__ __forceinline__ void phase_barrier()
{
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
}

// Step j on stage S for a wave of either half.  LEAD: waves 0..3.  PREV: the
// trailing half has a step j-1 to multiply (j > 0).
template <int S, int NMB, bool STREAM, bool LEAD, bool PREV>
__device__ __forceinline__ void pp_step(const Tile &t, const WaveConst &w, const Lds &l,
                                        f32x16 (&acc)[NMB > 0 ? NMB : 1][2], bf16x8 (&a0)[kHalfBlocks],
                                        bf16x8 (&a1)[kHalfBlocks], bf16x8 (&b0)[2], bf16x8 (&b1)[2], int j)
{
    // the fills of the kAhead - 1 steps after j are the loads issued after step j's
    constexpr int kAfter = (kAhead - 1) * (row_loads(NMB) + 2);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt((kAfter & 15) | ((kAfter >> 4) << 14) | (7 << 4) | (15 << 8));
    phase_barrier();                                        // E_j
    bf16 *fa = l.a((S + kAhead) & 3), *fb = l.b((S + kAhead) & 3);
    if constexpr (LEAD) {
        read_step<S, NMB>(w, l, a0, a1, b0, b1);
        phase_barrier();                                    // O_j
        mma_step<NMB, STREAM, true>(t, w, fa, fb, j + kAhead, acc, a0, a1, b0, b1);
    } else {
        if constexpr (PREV) mma_step<NMB, STREAM, true>(t, w, fa, fb, j + kAhead, acc, a0, a1, b0, b1);
        else fill<NMB, STREAM>(t, w, fa, fb, j + kAhead);
        phase_barrier();                                    // O_j
        read_step<S, NMB>(w, l, a0, a1, b0, b1);
        // the reads of stage S complete before E_{j+1}, where it is refilled
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4) | (0 << 8));
    }
}

// The tile for a wave whose half holds NMB row blocks (NMB = 0: the second
// half of a one-block tile; it loads no token rows and runs no MFMAs but
// fills its share of the weight fragments).  Both halves pass the same
// barriers.  row_h: tile row of the half's first block; col_w: the wave's
// first weight column; N: columns of the product.
template <int NMB, bool STREAM, bool LEAD, typename Request>
__device__ __forceinline__ void run_large(const Tile &t, const WaveConst &w, const Lds &l, const Out &o,
                                          int row_h, int col_w, int N, int lane, Request request)
{
    f32x16 acc[NMB > 0 ? NMB : 1][2];
#pragma unroll
    for (int i = 0; i < (NMB > 0 ? NMB : 1); ++i) acc[i][0] = acc[i][1] = (f32x16){};
    bf16x8 a0[kHalfBlocks], a1[kHalfBlocks], b0[2], b1[2];
    fill<NMB, STREAM>(t, w, l.a(0), l.b(0), 0);
    fill<NMB, STREAM>(t, w, l.a(1), l.b(1), 1);
    if constexpr (kAhead > 2) fill<NMB, STREAM>(t, w, l.a(2), l.b(2), 2);
    // K is a multiple of 128, so KT is a multiple of 4; the first step (the
    // trailing half has nothing to multiply yet), then branch-free bodies of
    // four steps (stage = step % 4)
    pp_step<0, NMB, STREAM, LEAD, false>(t, w, l, acc, a0, a1, b0, b1, 0);
    pp_step<1, NMB, STREAM, LEAD, true>(t, w, l, acc, a0, a1, b0, b1, 1);
    pp_step<2, NMB, STREAM, LEAD, true>(t, w, l, acc, a0, a1, b0, b1, 2);
    pp_step<3, NMB, STREAM, LEAD, true>(t, w, l, acc, a0, a1, b0, b1, 3);
    for (int j = 4; j < t.KT; j += 4) {
        pp_step<0, NMB, STREAM, LEAD, true>(t, w, l, acc, a0, a1, b0, b1, j);
        pp_step<1, NMB, STREAM, LEAD, true>(t, w, l, acc, a0, a1, b0, b1, j + 1);
        pp_step<2, NMB, STREAM, LEAD, true>(t, w, l, acc, a0, a1, b0, b1, j + 2);
        pp_step<3, NMB, STREAM, LEAD, true>(t, w, l, acc, a0, a1, b0, b1, j + 3);
    }
    // E_KT: the trailing half multiplies the last step
    phase_barrier();
    if constexpr (!LEAD) mma_step<NMB, STREAM, false>(t, w, nullptr, nullptr, 0, acc, a0, a1, b0, b1);
    __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));   // vmcnt(0): the look-ahead fills
    __syncthreads();                                     // landed before the ring is reused
    request();
    if constexpr (NMB > 0) {
        if (o.swiglu) {
            // row block mb of the half at h_stage(): 128 h columns a row
#pragma unroll
            for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) {
                    bf16 *p = h_stage(l, LEAD ? mb : kHalfBlocks + mb) + (lane & 31) * kHStride +
                              (w.wave & 3) * 32 + nb * 16 + (lane >> 5) * 8;
                    *(u32x4 *)p = h_block(acc[mb][nb]);
                }
        } else {
#pragma unroll
            for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
                    y_block(acc[mb][nb], o, row_h + mb * 32 + (lane & 31), col_w + nb * 32,
                            col_w + nb * 32 < N);
        }
    }
}

// The staged h of a large tile to memory: a block of 32 rows x 256 bytes is
// one 16-byte store of every thread.  nb0, nb: row blocks of the first half,
// of the tile; n0: the tile's first weight column.
__device__ __forceinline__ void store_h_large(const Lds &l, const Out &o, int nb0, int nb, int n0, int tid)
{
    __syncthreads();
    const int r = tid >> 4, c = tid & 15;
#pragma unroll
    for (int i = 0; i < kTileBlocks; ++i) {
        const int b = i < kHalfBlocks ? i : nb0 + i - kHalfBlocks;       // row block of the tile
        if (i < kHalfBlocks ? b >= nb0 : b >= nb) continue;
        const u32x4 v = *(const u32x4 *)(h_stage(l, i) + r * kHStride + c * 8);
        h_store(v, o, ((b * 32 + r) * o.ld + n0 / 2 + c * 8) * 2);
    }
}

template <bool STREAM, typename Request>
__device__ __forceinline__ void run_large_any(const Tile &t, const WaveConst &w, const Lds &l, const Out &o,
                                              int nmb, int row_h, int col_w, int N, int lane, Request request)
{
    if (w.wave < 4) {
        switch (nmb) {
        case 1: run_large<1, STREAM, true>(t, w, l, o, row_h, col_w, N, lane, request); break;
        case 2: run_large<2, STREAM, true>(t, w, l, o, row_h, col_w, N, lane, request); break;
        case 3: run_large<3, STREAM, true>(t, w, l, o, row_h, col_w, N, lane, request); break;
        case 4: run_large<4, STREAM, true>(t, w, l, o, row_h, col_w, N, lane, request); break;
        default: run_large<5, STREAM, true>(t, w, l, o, row_h, col_w, N, lane, request); break;
        }
    } else {
        switch (nmb) {
        case 0: run_large<0, STREAM, false>(t, w, l, o, row_h, col_w, N, lane, [] {}); break;
        case 1: run_large<1, STREAM, false>(t, w, l, o, row_h, col_w, N, lane, [] {}); break;
        case 2: run_large<2, STREAM, false>(t, w, l, o, row_h, col_w, N, lane, [] {}); break;
        case 3: run_large<3, STREAM, false>(t, w, l, o, row_h, col_w, N, lane, [] {}); break;
        case 4: run_large<4, STREAM, false>(t, w, l, o, row_h, col_w, N, lane, [] {}); break;
        default: run_large<5, STREAM, false>(t, w, l, o, row_h, col_w, N, lane, [] {}); break;
        }
    }
}

// ---------------------------------------------------------------------------
// Small tiles: all of a group's rows (up to kSmallRows) x 128 columns.
//
// With few rows per expert the product is bound by the weights' HBM stream.
// Every weight panel is read exactly once, non-temporally, straight from HBM
// into a 4-deep register ring; LDS carries only the token rows, in a 4-deep
// direct-to-LDS ring of 24 KB stages.  The eight waves form a 4 x 2 grid:
// wave (kq, ch) owns columns 64 ch .. + 63 of the tile and the K quarter
// [16 kq, + 16) of every 64-wide step, for all row blocks, so each token-row
// fragment is read from LDS by two waves only; the four K quarters are summed
// through LDS once per tile.  Every step issues the same loads (steps past K
// re-read the last one), so each step's wait is a constant.
// ---------------------------------------------------------------------------
constexpr int kBKs = 64;                 // bf16 per K step = 128 B per row

struct SmallTile {
    __amdgpu_buffer_rsrc_t ra, rb;
    int KT;
    int avoff[3];      // token-row load offsets of this lane's row groups wave + 8 i
    int vb;            // this lane's weight load offset in the 256-column panel (K step 0)
    int sstep;         // bytes of the panel per 64-wide K step
};

struct SmallWave {
    int wave, lane, kq, ch;
};

// Row group wave + 8 i (8 rows x 128 bytes) of step j into stage I.
template <int I>
__device__ __forceinline__ void fill_row(const SmallTile &t, const Lds &l, const SmallWave &w, int j, int i)
{
    const int js = min(j, t.KT - 1);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(t.ra, (lds_void *)(l.s[I] + (w.wave + 8 * i) * 8 * kBKs), 16,
                                             t.avoff[i], js * kBKs * 2, 0, 0);
}

// The wave's fragments of step j: its sub-step of column blocks 2 ch, 2 ch + 1.
template <int I>
__device__ __forceinline__ void fill_weights(const SmallTile &t, int j, bf16x8 (&breg)[4][2])
{
    const int soff = min(j, t.KT - 1) * t.sstep;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(t.rb, t.vb + c * 2048, soff, kNonTemporal);
        breg[I][c] = __builtin_bit_cast(bf16x8, v);
    }
}

// One K step with compile-time ring index I = k % 4: the step's two weight
// loads first (the HBM stream), then the token-row loads one at a time
// between the MFMAs; kRows + 2 loads per wave, all after the previous step's.
template <int NMB, int I>
__device__ __forceinline__ void small_step(const SmallTile &t, const Lds &l, const SmallWave &w,
                                           f32x16 (&acc)[NMB][2], int k, bf16x8 (&breg)[4][2])
{
    constexpr int kRows = (NMB + 1) / 2;           // row-group loads per wave and step
    constexpr int kAfter = 2 * (kRows + 2);        // the fills of steps k+1 and k+2
    __builtin_amdgcn_s_waitcnt((kAfter & 15) | ((kAfter >> 4) << 14) | (7 << 4) | (15 << 8));
    __builtin_amdgcn_s_barrier();          // every wave's fills of step k landed; step k-1 read
    fill_weights<(I + 3) & 3>(t, k + 3, breg);
    __builtin_amdgcn_sched_barrier(0);

    // Token-row fragment mb of sub-step kq: row 32 mb + lane % 32, 16-byte
    // chunk 2 kq + lane / 32, stored swizzled by (row / 2) % 8.
    const int rd_row = w.lane & 31;
    const int ch = ((2 * w.kq + (w.lane >> 5)) ^ ((rd_row >> 1) & 7)) << 3;
    const bf16 *As = l.s[I] + rd_row * kBKs + ch;
    bf16x8 af[NMB];
#pragma unroll
    for (int mb = 0; mb < NMB; ++mb) af[mb] = *(const bf16x8 *)&As[mb * 32 * kBKs];
    __builtin_amdgcn_sched_barrier(0);
    int nf = 0;
#pragma unroll
    for (int mb = 0; mb < NMB; ++mb) {
#pragma unroll
        for (int c = 0; c < 2; ++c)
            acc[mb][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(breg[I][c], af[mb], acc[mb][c], 0, 0, 0);
        if (nf < kRows) {
            fill_row<(I + 3) & 3>(t, l, w, k + 3, nf);
            ++nf;
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
}

template <int NMB, int I>
__device__ __forceinline__ void small_fill(const SmallTile &t, const Lds &l, const SmallWave &w, int j,
                                           bf16x8 (&breg)[4][2])
{
    fill_weights<I>(t, j, breg);
#pragma unroll
    for (int i = 0; i < (NMB + 1) / 2; ++i) fill_row<I>(t, l, w, j, i);
    __builtin_amdgcn_sched_barrier(0);
}

constexpr int kHStrideS = 64 + 8;         // staged h row of a small tile: 64 columns, padded

// The staged h of row blocks 2 r and 2 r + 1 to memory: 64 rows x 128 bytes,
// one 16-byte store of every thread.
__device__ __forceinline__ void small_store_h(const SmallWave &w, const Out &o, int n0, const bf16 *hst, int r)
{
    if (!o.swiglu) return;
    const int t = w.wave * 64 + w.lane, row = t >> 3, c = t & 7;
    h_store(*(const u32x4 *)(hst + row * kHStrideS + c * 8), o, ((r * 64 + row) * o.ld + n0 / 2 + c * 8) * 2);
}

// Sum of the K quarters and output of row blocks 2 R and 2 R + 1: every wave
// puts its partials (4 KB a block) into stage c = 2 (mb % 2) + column block,
// and wave (c, ch) sums the four quarters in order and writes the block.  All
// waves run the same instructions: a workgroup often runs one small tile of a
// launch, and then each line of this code is fetched from HBM.
template <int NMB, int R>
__device__ __forceinline__ void small_round(const Lds &l, const SmallWave &w, const f32x16 (&acc)[NMB][2],
                                            const Out &o, int n0, bf16 *hst)
{
    __syncthreads();                       // the stages are free, the last round's h is staged
    if constexpr (R > 0) small_store_h(w, o, n0, hst, R - 1);
    const int part = w.ch * 4 + w.kq;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        if (2 * R + (c >> 1) >= NMB) continue;
        const f32x16 &v = acc[2 * R + (c >> 1) < NMB ? 2 * R + (c >> 1) : 0][c & 1];
        f32x4 *p = (f32x4 *)(l.s[c] + part * 2048) + w.lane;
#pragma unroll
        for (int g = 0; g < 4; ++g) p[g * 64] = (f32x4){v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
    }
    __syncthreads();
    const int mb = 2 * R + (w.kq >> 1), tok = (w.kq >> 1) * 32 + (w.lane & 31);
    if (mb < NMB) {
        const bf16 *st = w.kq == 0 ? l.s[0] : w.kq == 1 ? l.s[1] : w.kq == 2 ? l.s[2] : l.s[3];
        const f32x4 *p = (const f32x4 *)(st + w.ch * 4 * 2048) + w.lane;
        f32x16 v;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            f32x4 x = p[g * 64];
#pragma unroll
            for (int q = 1; q < 4; ++q) {
                const f32x4 y = p[q * 256 + g * 64];
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] += y[e];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * g + e] = x[e];
            __builtin_amdgcn_sched_barrier(0);
        }
        if (o.swiglu)
            *(u32x4 *)(hst + tok * kHStrideS + w.ch * 32 + (w.kq & 1) * 16 + (w.lane >> 5) * 8) = h_block(v);
        else
            y_block(v, o, R * 64 + tok, n0 + w.ch * 64 + (w.kq & 1) * 32, true);
    }
}

template <int NMB>
__device__ __forceinline__ void small_finish(const Lds &l, const SmallWave &w, const f32x16 (&acc)[NMB][2],
                                             const Out &o, int n0, bf16 *hst)
{
    small_round<NMB, 0>(l, w, acc, o, n0, hst);
    if constexpr (NMB > 2) small_round<NMB, 1>(l, w, acc, o, n0, hst);
    if constexpr (NMB > 4) small_round<NMB, 2>(l, w, acc, o, n0, hst);
    __syncthreads();
    small_store_h(w, o, n0, hst, (NMB - 1) / 2);
}

// One tile with NMB 32-row blocks: K loop, sum of the K quarters and
// epilogue, fully unrolled over the row blocks so no accumulator crosses a
// branch.  n0: the tile's first weight column.
template <int NMB, typename Request>
__device__ __forceinline__ void run_small(const SmallTile &t, const Lds &l, const SmallWave &w,
                                          const Out &o, int n0, bf16 *hst, Request request)
{
    f32x16 acc[NMB][2];
#pragma unroll
    for (int i = 0; i < NMB; ++i) acc[i][0] = acc[i][1] = (f32x16){};
    bf16x8 breg[4][2];
    small_fill<NMB, 0>(t, l, w, 0, breg);
    small_fill<NMB, 1>(t, l, w, 1, breg);
    small_fill<NMB, 2>(t, l, w, 2, breg);
    // K is a multiple of 128, so KT is even: groups of 4 steps, then 2.
    int k = 0;
    for (; k + 4 <= t.KT; k += 4) {
        small_step<NMB, 0>(t, l, w, acc, k, breg);
        small_step<NMB, 1>(t, l, w, acc, k + 1, breg);
        small_step<NMB, 2>(t, l, w, acc, k + 2, breg);
        small_step<NMB, 3>(t, l, w, acc, k + 3, breg);
    }
    if (k < t.KT) {
        small_step<NMB, 0>(t, l, w, acc, k, breg);
        small_step<NMB, 1>(t, l, w, acc, k + 1, breg);
    }
    // The look-ahead fills (clamped re-reads of the last step) may still be
    // landing in the ring, which the partials overwrite next.
    __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));   // vmcnt(0)
    request();
    small_finish<NMB>(l, w, acc, o, n0, hst);
}

// Tiles of more than 160 rows: the accumulators of the 4 x 2 grid do not fit
// the registers, so the waves form a 2 x 4 grid instead: wave (kh, cq) owns
// columns 32 cq .. + 31 and the K half [32 kh, + 32) of every step (twice the
// LDS reads for the same tile).  The weight loads are the wave's two sub-steps
// of its column block.
constexpr int kTallBlocks = 6;

template <int I>
__device__ __forceinline__ void fill_weights_tall(const SmallTile &t, int j, bf16x8 (&breg)[4][2])
{
    const int soff = min(j, t.KT - 1) * t.sstep;
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(t.rb, t.vb + m * 1024, soff, kNonTemporal);
        breg[I][m] = __builtin_bit_cast(bf16x8, v);
    }
}

template <int I>
__device__ __forceinline__ void tall_step(const SmallTile &t, const Lds &l, const SmallWave &w,
                                          f32x16 (&acc)[kTallBlocks], int k, bf16x8 (&breg)[4][2])
{
    constexpr int NMB = kTallBlocks, kRows = NMB / 2, kAfter = 2 * (kRows + 2);
    __builtin_amdgcn_s_waitcnt((kAfter & 15) | ((kAfter >> 4) << 14) | (7 << 4) | (15 << 8));
    __builtin_amdgcn_s_barrier();
    fill_weights_tall<(I + 3) & 3>(t, k + 3, breg);
    __builtin_amdgcn_sched_barrier(0);
    const int rd_row = w.lane & 31, swz = (rd_row >> 1) & 7, kh = w.wave >> 2;
    bf16x8 af[2][NMB];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int mb = 0; mb < NMB; ++mb)
            af[m][mb] = *(const bf16x8 *)&l.s[I][(mb * 32 + rd_row) * kBKs +
                                                 (((4 * kh + 2 * m + (w.lane >> 5)) ^ swz) << 3)];
    __builtin_amdgcn_sched_barrier(0);
    int nf = 0;
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int mb = 0; mb < NMB; ++mb) {
            acc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(breg[I][m], af[m][mb], acc[mb], 0, 0, 0);
            if (nf < kRows && (m * NMB + mb) % 2 == 0) {
                fill_row<(I + 3) & 3>(t, l, w, k + 3, nf);
                ++nf;
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    __builtin_amdgcn_sched_barrier(0);
}

template <int I>
__device__ __forceinline__ void tall_fill(const SmallTile &t, const Lds &l, const SmallWave &w, int j,
                                          bf16x8 (&breg)[4][2])
{
    fill_weights_tall<I>(t, j, breg);
#pragma unroll
    for (int i = 0; i < kTallBlocks / 2; ++i) fill_row<I>(t, l, w, j, i);
    __builtin_amdgcn_sched_barrier(0);
}

// K-half partials of row block mb, column block cq: 4 KB at 4 KB (4 (mb / 4) +
// cq) of stage mb % 4; wave (kh, cq) finishes the blocks with mb % 2 = kh.
template <int KH>
__device__ __forceinline__ void tall_finish(const Lds &l, const SmallWave &w, const f32x16 (&acc)[kTallBlocks],
                                            const Out &o, int col)
{
    const int cq = w.wave & 3;
#pragma unroll
    for (int mb = 1 - KH; mb < kTallBlocks; mb += 2) {
        f32x4 *part = (f32x4 *)(l.s[mb & 3] + ((mb >> 2) * 4 + cq) * 2048) + w.lane;
#pragma unroll
        for (int g = 0; g < 4; ++g)
            part[g * 64] = (f32x4){acc[mb][4 * g], acc[mb][4 * g + 1], acc[mb][4 * g + 2], acc[mb][4 * g + 3]};
    }
    __syncthreads();
#pragma unroll
    for (int mb = KH; mb < kTallBlocks; mb += 2) {
        f32x16 v = acc[mb];
        const f32x4 *part = (const f32x4 *)(l.s[mb & 3] + ((mb >> 2) * 4 + cq) * 2048) + w.lane;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f32x4 p = part[g * 64];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * g + e] += p[e];
        }
        const int tok = mb * 32 + (w.lane & 31);
        if (o.swiglu) h_store(h_block(v), o, (tok * o.ld + col / 2 + (w.lane >> 5) * 8) * 2);
        else y_block(v, o, tok, col, true);
    }
}

template <typename Request>
__device__ __forceinline__ void run_tall(const SmallTile &t, const Lds &l, const SmallWave &w, const Out &o,
                                         int col, Request request)
{
    f32x16 acc[kTallBlocks];
#pragma unroll
    for (int i = 0; i < kTallBlocks; ++i) acc[i] = (f32x16){};
    bf16x8 breg[4][2];
    tall_fill<0>(t, l, w, 0, breg);
    tall_fill<1>(t, l, w, 1, breg);
    tall_fill<2>(t, l, w, 2, breg);
    int k = 0;
    for (; k + 4 <= t.KT; k += 4) {
        tall_step<0>(t, l, w, acc, k, breg);
        tall_step<1>(t, l, w, acc, k + 1, breg);
        tall_step<2>(t, l, w, acc, k + 2, breg);
        tall_step<3>(t, l, w, acc, k + 3, breg);
    }
    if (k < t.KT) {
        tall_step<0>(t, l, w, acc, k, breg);
        tall_step<1>(t, l, w, acc, k + 1, breg);
    }
    __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));   // vmcnt(0): look-ahead fills
    request();
    __syncthreads();
    if (w.wave < 4) tall_finish<0>(l, w, acc, o, col); else tall_finish<1>(l, w, acc, o, col);
}

}  // namespace

template <bool LARGE>
__global__ __launch_bounds__(kThreads, 1)
void k_ffn_bf16(FfnArgs)
{
    KernArgs args = kernel_args();
    __shared__ __attribute__((aligned(1024))) bf16 lds_0[kStageElems];
    __shared__ __attribute__((aligned(1024))) bf16 lds_1[kStageElems];
    __shared__ __attribute__((aligned(1024))) bf16 lds_2[kStageElems];
    __shared__ __attribute__((aligned(1024))) bf16 lds_3[kStageElems];
    __shared__ __attribute__((aligned(16))) bf16 lds_h[64 * kHStrideS];
    __shared__ SchedLds sl;
    const Lds l{{lds_0, lds_1, lds_2, lds_3}};

    int tid = threadIdx.x;
    Worker<LARGE> wk;
    if (tid == 192) {                     // the layer's weights, while begin() loads
        const void *W1 = args->p1.W, *W2 = args->p2.W;
        if (args->layer_id) {
            int ly = *args->layer_id;
            if (ly < 0 || ly >= args->n_layers) {
                if (blockIdx.x == 0 && args->sched.hdr[0] > 0) atomicOr(args->err, kErrBadLayer);
                ly = ly < 0 ? 0 : args->n_layers - 1;
            }
            W1 = args->layers[ly].w1;
            W2 = args->layers[ly].w2;
        }
        sl.w[0] = (uint64_t)W1;
        sl.w[1] = (uint64_t)W2;
    }
    if (!wk.begin(args->sched, sl, args->phases, args->tiles)) return;

    for (;;) {
        args = reload(args);
        asm volatile("" : "+v"(tid));
        if (!wk.next(args->sched, sl, args->phases, args->tiles, args->err)) break;
        args = reload(args);
        // nothing that a lane derives from its number is kept over the items
        asm volatile("" : "+v"(tid));
        const int lane = tid & 63;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const bool down = wk.down;
        auto request = [&] { wk.request(); };
        const RowTile rt = wk.row_tile(args->sched, sl);
        const bool sh = rt.group == args->shared_group;
        const int N = down ? args->p2.N : args->p1.N, K = down ? args->p2.K : args->p1.K;
        const void *Ar = down ? args->p2.A_routed : args->p1.A_routed, *As = down ? args->p2.A_shared : args->p1.A_shared;
        void *Cr = down ? args->p2.C_routed : args->p1.C_routed, *Cs = down ? args->p2.C_shared : args->p1.C_shared;
        const int32_t *index = (!down && !sh) ? args->A_index : nullptr;
        const bf16 *A = index ? (const bf16 *)Ar : (const bf16 *)(sh ? As : Ar) + (int64_t)rt.row0 * K;
        const __amdgpu_buffer_rsrc_t ra = make_rsrc(A, (index ? args->A_routed_rows : (int64_t)rt.rows) * K * 2);
        Out o;
        o.ld = down ? args->p2.ldc : args->p1.ldc;
        o.swiglu = !down;
        o.r = make_rsrc((bf16 *)(sh ? Cs : Cr) + (int64_t)rt.row0 * o.ld, (int64_t)rt.rows * o.ld * 2);
        const bf16 *W = uniform_ptr((const bf16 *)sl.w[down ? 1 : 0]);
        const int nb = (rt.rows + 31) >> 5;
        if (LARGE && wk.large) {
            const int n0 = wk.nt * 256;
            WaveConst w;
            w.wave = wave;
            w.voff_b = lane * 16;
            const int rd_row = lane & 31;
            w.rd_hi = lane >> 5;
            w.swz = (rd_row >> 2) & 3;
            w.a_rd = ((wave >> 2) * kHalfRows + rd_row) * kRowElems;
            w.b_rd = ((wave & 3) * 2) * 2 * 512 + lane * 8;
            Tile t;
            t.ra = ra;
            t.KT = K / kBK;
            t.ncb = min(256, N - n0) / 32;
            t.stepb = t.ncb * 2048;
            // the tile's column blocks n0/32 .. are one panel, contiguous
            t.rb = make_rsrc(W + ((int64_t)rt.group * N + n0) * K, (int64_t)t.ncb * 32 * K * 2);
            const int nb0 = (nb + 1) >> 1;               // row blocks of the first half
            const int nmb = wave < 4 ? nb0 : nb - nb0;
            const int row_h = wave < 4 ? 0 : nb0 * 32;   // tile row of this wave's half
            {
                // token fill: waves w and w + 4 load row groups w % 4, 4 + w % 4
                // and 8 + w % 2 (16 rows each; groups 8 and 9 are loaded twice,
                // to the same place) of their half; lane l covers row l / 4,
                // chunk l % 4, and (row / 4) % 4 = (l / 16) % 4.  Rows past the
                // half or the tile get an offset past every buffer range and
                // read as zero.
                const int chunk = ((lane & 3) ^ ((lane >> 4) & 3)) << 4;
                const int hrows = min(rt.rows - row_h, nmb * 32);
                int src[3], hr[3];
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const int g = i < 2 ? (wave & 3) + 4 * i : 8 + (wave & 1);
                    w.a_wr[i] = ((wave >> 2) * kHalfRows + g * 16) * kRowElems;
                    hr[i] = g * 16 + (lane >> 2);
                    const int r = min(hr[i], max(hrows - 1, 0)) + (hrows > 0 ? row_h : 0);
                    src[i] = index ? index[rt.row0 + r] / args->A_index_div : r;
                }
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    t.va[i] = hr[i] < hrows ? src[i] * K * 2 + chunk : (int)0x80000000u;
            }
            const int col_w = n0 + (wave & 3) * 64;
            if (rt.only) run_large_any<true>(t, w, l, o, nmb, row_h, col_w, N, lane, request);
            else run_large_any<false>(t, w, l, o, nmb, row_h, col_w, N, lane, request);
            if (o.swiglu) store_h_large(l, o, nb0, nb, n0, tid);
        } else {
            const int n0 = wk.nt * 128;
            SmallWave sw{wave, lane, wave >> 1, wave & 1};
            SmallTile t;
            t.ra = ra;
            t.KT = K / kBKs;
            // the tile is one half of a 256-column panel, which holds per
            // 32-wide K step its ncb column blocks' two 1 KB fragments
            // contiguously; wave (kq, ch) reads sub-step kq % 2 of column blocks
            // 4 half + 2 ch and + 1 of the panel's K step 2 js + kq / 2
            const int p0 = n0 & ~255, half = (n0 >> 7) & 1;
            const int ncb = min(8, (N - p0) / 32);
            t.rb = make_rsrc(W + ((int64_t)rt.group * N + p0) * K, (int64_t)ncb * 32 * K * 2);
            t.sstep = ncb * 4096;
            t.vb = (sw.kq >> 1) * ncb * 2048 + (4 * half + 2 * sw.ch) * 2048 + (sw.kq & 1) * 1024 + lane * 16;
            // lane l of a row-group load covers row 8 rg + l / 8, physical chunk
            // l % 8 <- global chunk (l % 8) ^ ((row / 2) % 8); rows past the
            // group get an offset past every buffer range and read as zero
            int src[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const int r = min(8 * (wave + 8 * i) + (lane >> 3), rt.rows - 1);
                src[i] = index ? index[rt.row0 + r] / args->A_index_div : r;
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const int r = 8 * (wave + 8 * i) + (lane >> 3);
                t.avoff[i] = r < rt.rows ? src[i] * K * 2 + (((lane & 7) ^ ((r >> 1) & 7)) << 4)
                                         : (int)0x80000000u;
            }
            if (nb == kTallBlocks) {
                t.vb = (wave >> 2) * ncb * 2048 + (4 * half + (wave & 3)) * 2048 + lane * 16;
                run_tall(t, l, sw, o, n0 + (wave & 3) * 32, request);
            } else switch (nb) {
            case 1: run_small<1>(t, l, sw, o, n0, lds_h, request); break;
            case 2: run_small<2>(t, l, sw, o, n0, lds_h, request); break;
            case 3: run_small<3>(t, l, sw, o, n0, lds_h, request); break;
            case 4: run_small<4>(t, l, sw, o, n0, lds_h, request); break;
            default: run_small<5>(t, l, sw, o, n0, lds_h, request); break;
            }
        }
        args = reload(args);
        wk.done(args->sched, sl, args->phases, args->tiles);
    }
}

}  // namespace moe
