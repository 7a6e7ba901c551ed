// e4m3 grouped GEMM with DeepSeek-style block scaling (fp8 variant of the
// expert stage): activations carry one fp32 scale per row and 128-channel
// group, weights one fp32 scale per 128x128 block.  Each K step covers
// exactly one 128-wide scale group g:
//
//   t    = sum over the group of e4m3(W) * e4m3(X)     (v_mfma 16x16x128 f8)
//   acc += t * (s_X[token, g] * s_W[block, g])          (fp32 promotion)
//
// so the block scales are applied exactly once per group in fp32.  The
// hardware's per-32-element power-of-two (E8M0) MFMA scales cannot express
// these fp32 scales and are left at 1.
//
// Design for gfx950:
//  * one persistent workgroup per CU runs items (128-token x 256-feature
//    tiles) of both products in one launch (or in one each, split_products()),
//    from the lists of ffn_sched.h: a down item starts once the gate/up tiles of its rows are written, so no
//    idle last round and no launch gap lies between the products (T = 32768,
//    d = 7168, f = 2048, 8 experts, with dispatch and combine: 539 -> 497 us;
//    T = 2049: 132 -> 126).  Row tiles are rastered in bands of up to 8 so that each weight
//    panel is read by one XCD;
//  * the product is formed transposed, D[feature][token] = W X^T: the
//    weights are the MFMA's row operand and the tokens its column operand,
//    so each lane holds four consecutive features of ONE token and the
//    token's fp32 scale is a single value per lane and 16-token block;
//  * eight wave64s, wave w owning features 64 (w % 4) .. + 63 and tokens
//    64 (w / 4) .. + 63 of the tile as 4 x 4 blocks of
//    v_mfma_scale_f32_16x16x128_f8f6f4; the two waves of a SIMD (w and
//    w + 4) work in opposite phases, one reading its operands from LDS
//    while the other runs its MFMAs and promotion (the K loop below);
//  * K advances one scale group (128 bytes) per step through a 3-deep LDS
//    ring of 48.5 KB stages (32 KB of weight fragments, 16 KB of token rows,
//    the step's 128 token scales) filled by direct-to-LDS buffer loads two
//    groups ahead: every group issues the same seven loads per wave, so the
//    wait before a group is the constant vmcnt(7) (the next group's fills
//    stay in flight) and no wait drains the look-ahead.  The loads go out
//    one by one between the MFMAs: a stage is 49 loads of 1 KB per CU, about
//    as many clocks of the per-CU load path as the group's MFMAs take, and
//    issued as one burst they held back every wave's instructions;
//  * the weights are packed in the 16 x 128 fragment order of the MFMA (two
//    lane-contiguous 1 KB halves per fragment), gate and up rows interleaved
//    by 16, so each wave's 64 features are gate and up rows of the same 32 h
//    channels (one scalar scale each per group: the gate and the up 128 x 128
//    block) and a 256-feature gate/up tile covers exactly one 128-channel
//    group of h;
//  * token rows are 128-byte rows whose 16-byte chunks are XOR-swizzled by
//    (row / 2) & 5: a lane reads two chunks 4 apart, and with this mask neither
//    read has a bank conflict ((row / 2) % 8 has: 1% of the time at T = 32768
//    and above); rows past a group's end have an offset past every buffer
//    range and read as zero; the scalar offset, which the range check does
//    not cover, only moves along K (clamped to the last group) and between
//    weight fragments that exist;
//  * the gate/up product reads the routed token rows straight from x through
//    slot_of_row (the row gather is part of the token fills, as in bf16); the
//    rows' fp32 scales arrive already gathered and transposed, one
//    contiguous run of 128 per group, since reading them per token would cost
//    one cache line per lane and load;
//  * SwiGLU mode: every wave forms h = SiLU(gate) * up in fp32 for its 32
//    channels, the per-token |h| maximum over the tile's 128 channels meets
//    in a 2 KB LDS table, and each token's channels are quantised to e4m3
//    with one fp32 scale amax / 448 (the activation quantiser's scale;
//    the quotient is taken as a product with the scale's reciprocal).  The
//    codes are staged in LDS and leave as whole 128-byte rows, past this XCD's
//    L2 to memory (the down items that read them run on other XCDs in the same
//    launch).  The down product reads the rows' scales the same way (the gate/up
//    product's scales are inputs and keep ordinary loads: 0.7% of the time) and
//    writes bf16, four
//    consecutive features per lane.
#include "ffn_sched.h"
#include "kernels.h"

namespace moe {

namespace {

constexpr int kGrpB = 128;                   // K bytes per step: one scale group
constexpr int kTokT = 128;                   // tokens per tile
constexpr int kFeatT = 256;                  // features per tile
constexpr int kWBytes = kFeatT * kGrpB;      // weight fragments of one stage: 32 KB
constexpr int kXBytes = kTokT * kGrpB;       // token rows of one stage: 16 KB
constexpr int kXSBytes = kXBytes + kTokT * 4; // ... followed by the step's 128 token scales
constexpr int kWaves8 = 8;
constexpr int kThreads8 = 64 * kWaves8;
constexpr int kHStride8 = 128 + 16;          // staged h codes: a row of 128, padded
constexpr int kAgentScope8 = 16;             // sc1: past this XCD's L2
static_assert(kTokT == 32 * kTileBlocksFp8, "row tiles of the schedule");
static_assert(kTokT * kHStride8 <= kWBytes, "the staged codes fit one stage's weights");
constexpr int kFillLoads = 7;                // loads per wave per group fill
typedef __attribute__((address_space(3))) void lds_void;

// 16-byte chunks of LDS token row r are XOR-swizzled by this.
__device__ __forceinline__ int x_swizzle(int r) { return (r >> 1) & 5; }

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc8(const void *base, int64_t bytes)
{
    int32_t n = bytes > 0x7fffffff ? 0x7fffffff : (int32_t)bytes;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, n, 0x00020000);
}

// Weight scales are read-only while a GEMM runs: reading them through the
// constant address space makes the per-group read a scalar load, which
// neither waits for nor counts against the in-flight direct-to-LDS fills (a
// flat load may alias LDS, so the compiler would drain the fills before it).
typedef const __attribute__((address_space(4))) float cfloat;

struct Tile8 {
    __amdgpu_buffer_rsrc_t rw, rx, rs;
    int vx[2];          // token fills: rows 16 w + 8 i + lane / 8, swizzled chunk (or past the range)
    int KT, ncb, cbstride, s_ld;
    const cfloat *sbp0; // weight scale of each K group: feature blocks rb = 0, 2 of this wave
    const cfloat *sbp1; //   ... and rb = 1, 3 (in SwiGLU mode the up rows; otherwise = sbp0)
};

struct Ring8 {
    uint8_t *w, *x;
    float *s;
};

// Fills of K group kg (clamped to the last) into one stage, 7 loads per wave:
//  * weight fragments 2 w and 2 w + 1 of the tile's 16, both 1 KB halves;
//  * token rows 16 w .. 16 w + 15 as two 8-row instructions; lane l writes
//    LDS row 16 w + 8 i + l / 8, physical chunk l % 8, with global chunk
//    (l % 8) ^ ((row / 2) & 5);
//  * 64 of the 128 token scales (waves w and w + 2, w + 4, w + 6 load the
//    same ones: identical data to identical addresses).
// Load i (0..6) of the fills: 0..3 the weight fragment halves, 4..5 the
// token rows, 6 the token scales.
template <bool DOWN>
__device__ __forceinline__ void fill8_one(const Tile8 &t, const Ring8 &st, int wave, int lane, int kg,
                                          int i)
{
    const int ks = min(kg, t.KT - 1);
    if (i < 4) {
        const int f = wave * 2 + (i >> 1), h = i & 1;
        const int cb = min(f, t.ncb - 1);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(t.rw, (lds_void *)(st.w + f * 2048 + h * 1024), 16,
                                                 lane * 16, cb * t.cbstride + ks * 2048 + h * 1024,
                                                 0, 0);
    } else if (i < 6) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(t.rx, (lds_void *)(st.x + (wave * 16 + (i - 4) * 8) * kGrpB),
                                                 16, t.vx[i - 4], ks * kGrpB, 0, 0);
    } else {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(t.rs, (lds_void *)(st.s + (wave & 1) * 64), 4,
                                                 (ks * t.s_ld + (wave & 1) * 64 + lane) * 4, 0, 0,
                                                 DOWN ? kAgentScope8 : 0);
    }
}

template <bool DOWN>
__device__ __forceinline__ void fill8(const Tile8 &t, const Ring8 &st, int wave, int lane, int kg)
{
#pragma unroll
    for (int i = 0; i < kFillLoads; ++i) fill8_one<DOWN>(t, st, wave, lane, kg, i);
}

struct Wave8 {
    int wave, lane, wf, wt;
    int w_rd;           // LDS byte offset of this lane's weight chunk (feature block 0)
    int x_rd0, x_rd1;   // LDS byte offsets of this lane's two token chunks (token block 0)
    int s_rd;           // LDS float index of this lane's token scale (token block 0)
};

// The K loop runs two waves per SIMD in opposite phases ("ping-pong"):
// waves 0..3 (tokens 0..63 of the tile) read group g's operands from LDS
// while waves 4..7 (tokens 64..127) run group g-1's MFMAs, and at the next
// barrier the roles swap, so one wave's LDS reads run under the other's
// matrix-core work instead of every wave reading, then every wave
// multiplying.  In slots E_g, O_g (one barrier before each):
//
//   slot   waves 0..3          waves 4..7
//   E_g    read g              MFMAs of g-1
//   O_g    MFMAs of g          read g
//
// Every wave issues its fills of group g+2 at the start of E_g, into the
// stage of group g-1, which waves 0..3 read in E_{g-1} (and consumed in
// O_{g-1}) and waves 4..7 in O_{g-1} (and waited for before E_g).  Before
// the barrier that starts E_g each wave waits for its own fills of g; only
// those of g+1 (seven loads) stay in flight.

// LDS reads of group g from stage S into registers: the four weight
// fragments, the NCB token fragments and their token scales.  The previous
// group's last token block is promoted here, under the reads' latency.
template <int S, int NCB>
__device__ __forceinline__ void read8(const Wave8 &w, const Ring8 (&ring)[3], i32x8 (&wfr)[4],
                                      i32x8 (&xf)[4], float (&st)[4], f32x4 (&acc)[4][4],
                                      const f32x4 (&pend)[4], const float (&ps)[2])
{
    if constexpr (NCB > 0) {
        const uint8_t *Ws = ring[S].w;
        const uint8_t *Xs = ring[S].x;
        const float *Ss = ring[S].s;
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) {
            const i32x4 lo = *(const i32x4 *)&Ws[w.w_rd + rb * 2048];
            const i32x4 hi = *(const i32x4 *)&Ws[w.w_rd + rb * 2048 + 1024];
            wfr[rb] = (i32x8){lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        }
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
            const i32x4 lo = *(const i32x4 *)&Xs[w.x_rd0 + cb * 16 * kGrpB];
            const i32x4 hi = *(const i32x4 *)&Xs[w.x_rd1 + cb * 16 * kGrpB];
            xf[cb] = (i32x8){lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            st[cb] = Ss[w.s_rd + cb * 16];
        }
#pragma unroll
        for (int rb = 0; rb < 4; ++rb)
            acc[rb][NCB - 1] = pend[rb] * ps[rb & 1] + acc[rb][NCB - 1];
    }
}

// The 4 x NCB MFMAs of one group, each token block's products promoted
// (acc += t * s_X * s_W) while the next block's MFMAs run; the last block's
// products are left in pend with their scales in ps.  The wave's seven fill
// loads of group kgf go out two per token block, after its second and fourth
// MFMA (the rest after the last MFMA when NCB < 4): the per-CU load path
// accepts about one 1 KB load every 19 clocks, and fills issued as one burst
// by every wave hold each wave's later instructions until the load path has
// taken them.
template <int NCB, bool DOWN, bool FILL = true>
__device__ __forceinline__ void mfma8(const i32x8 (&wfr)[4], const i32x8 (&xf)[4],
                                      const float (&st)[4], float sb0, float sb1,
                                      f32x4 (&acc)[4][4], f32x4 (&pend)[4], float (&ps)[2],
                                      const Tile8 &t, const Ring8 &fst, int wave, int lane, int kgf)
{
    constexpr int kInter = !FILL ? 0 : (2 * NCB < kFillLoads) ? 2 * NCB : kFillLoads;
    if constexpr (NCB > 0) {
        f32x4 tq[2][4];
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
            // one token block: its four MFMAs with two fill loads, and the
            // previous block's promotion, in a fixed issue order (one MFMA,
            // then four promotion instructions, while the MFMA holds the
            // matrix core for 32 cycles)
#pragma unroll
            for (int rb = 0; rb < 4; ++rb) {
                const f32x4 p = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
                    wfr[rb], xf[cb], (f32x4){}, 0, 0, 0, 127, 0, 127);
                if (cb == NCB - 1) pend[rb] = p; else tq[cb & 1][rb] = p;
                const int j = 2 * cb + (rb >> 1);
                if ((rb & 1) && j < kInter) fill8_one<DOWN>(t, fst, wave, lane, kgf, j);
            }
            if (cb > 0) {
                const float s0 = st[cb - 1] * sb0, s1 = st[cb - 1] * sb1;
#pragma unroll
                for (int rb = 0; rb < 4; ++rb)
                    acc[rb][cb - 1] = tq[(cb - 1) & 1][rb] * ((rb & 1) ? s1 : s0) + acc[rb][cb - 1];
            }
#pragma unroll
            for (int rb = 0; rb < 4; ++rb) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                        // MFMA
                if (cb > 0) __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);           // VALU
                if ((rb & 1) && 2 * cb + (rb >> 1) < kInter)
                    __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);                    // VMEM
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        ps[0] = st[NCB - 1] * sb0;
        ps[1] = st[NCB - 1] * sb1;
    }
#pragma unroll
    for (int i = kInter; i < (FILL ? kFillLoads : 0); ++i) fill8_one<DOWN>(t, fst, wave, lane, kgf, i);
}

// s_waitcnt operands (gfx9 encoding: vmcnt [3:0] and [15:14], expcnt [6:4],
// lgkmcnt [11:8]).
constexpr int kWaitFills = (kFillLoads & 15) | ((kFillLoads >> 4) << 14) | (7 << 4) | (15 << 8);
constexpr int kWaitLds = 15 | (3 << 14) | (7 << 4) | (0 << 8);

// A slot boundary, with the wait before it: the scheduler moves nothing
// across it (a wait drawn into the slot before it would shorten the
// fills' look-ahead).
template <int WAIT>
__device__ __forceinline__ void slot_barrier()
{
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (WAIT >= 0) __builtin_amdgcn_s_waitcnt(WAIT);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
}

// Group g (stage S) for a wave of either half.  LEAD: waves 0..3.  MFMA_PREV:
// the trailing half has a group g-1 to multiply (g > 0).
template <int S, int NCB, bool LEAD, bool DOWN, bool MFMA_PREV>
__device__ __forceinline__ void group8(const Tile8 &t, const Wave8 &w, const Ring8 (&ring)[3],
                                       f32x4 (&acc)[4][4], i32x8 (&wfr)[4], i32x8 (&xf)[4],
                                       float (&st)[4], float (&sb)[2], float (&sb_next)[2],
                                       f32x4 (&pend)[4], float (&ps)[2], int kg)
{
    slot_barrier<kWaitFills>();                   // E_kg, after this wave's fills of group kg
    const Ring8 &fst = ring[(S + 2) % 3];         // group kg+2's stage, read last by group kg-1
    if constexpr (LEAD) {
        sb[0] = sb_next[0];
        sb[1] = sb_next[1];
        sb_next[0] = t.sbp0[min(kg + 1, t.KT - 1)];
        sb_next[1] = t.sbp1[min(kg + 1, t.KT - 1)];
        read8<S, NCB>(w, ring, wfr, xf, st, acc, pend, ps);
        slot_barrier<-1>();                       // O_kg
        mfma8<NCB, DOWN>(wfr, xf, st, sb[0], sb[1], acc, pend, ps, t, fst, w.wave, w.lane, kg + 2);
    } else {
        if constexpr (MFMA_PREV)
            mfma8<NCB, DOWN>(wfr, xf, st, sb[0], sb[1], acc, pend, ps, t, fst, w.wave, w.lane, kg + 2);
        else
            fill8<DOWN>(t, fst, w.wave, w.lane, kg + 2);
        slot_barrier<-1>();                       // O_kg
        sb[0] = sb_next[0];
        sb[1] = sb_next[1];
        sb_next[0] = t.sbp0[min(kg + 1, t.KT - 1)];
        sb_next[1] = t.sbp1[min(kg + 1, t.KT - 1)];
        read8<S, NCB>(w, ring, wfr, xf, st, acc, pend, ps);
        // the reads of stage S complete before E_{kg+1}, where it is refilled
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(kWaitLds);
    }
}

// The K loop of one tile for a wave of one half with NCB token blocks
// holding tokens.  Both halves pass 2 KT + 1 barriers.
template <bool LEAD, int NCB, bool DOWN>
__device__ __forceinline__ void kloop8(const Tile8 &t, const Wave8 &w, const Ring8 (&ring)[3],
                                       f32x4 (&acc)[4][4])
{
    float sb[2] = {0.0f, 0.0f};
    float sb_next[2] = {t.sbp0[0], t.sbp1[0]};
    f32x4 pend[4] = {};
    float ps[2] = {0.0f, 0.0f};
    i32x8 wfr[4], xf[4];
    float st[4];
    __builtin_amdgcn_sched_barrier(0);
    fill8<DOWN>(t, ring[0], w.wave, w.lane, 0);
    fill8<DOWN>(t, ring[1], w.wave, w.lane, 1);
    // the first group (the trailing half has nothing to multiply yet), a
    // branch-free body of three groups (stage = group % 3), then the rest
    group8<0, NCB, LEAD, DOWN, false>(t, w, ring, acc, wfr, xf, st, sb, sb_next, pend, ps, 0);
    int kg = 1;
    for (; kg + 3 <= t.KT; kg += 3) {
        group8<1, NCB, LEAD, DOWN, true>(t, w, ring, acc, wfr, xf, st, sb, sb_next, pend, ps, kg);
        group8<2, NCB, LEAD, DOWN, true>(t, w, ring, acc, wfr, xf, st, sb, sb_next, pend, ps, kg + 1);
        group8<0, NCB, LEAD, DOWN, true>(t, w, ring, acc, wfr, xf, st, sb, sb_next, pend, ps, kg + 2);
    }
    if (kg < t.KT) group8<1, NCB, LEAD, DOWN, true>(t, w, ring, acc, wfr, xf, st, sb, sb_next, pend, ps, kg);
    if (kg + 1 < t.KT) group8<2, NCB, LEAD, DOWN, true>(t, w, ring, acc, wfr, xf, st, sb, sb_next, pend, ps, kg + 1);
    // E_KT: the trailing half multiplies the last group
    slot_barrier<-1>();
    if constexpr (!LEAD)
        mfma8<NCB, DOWN, false>(wfr, xf, st, sb[0], sb[1], acc, pend, ps, t, ring[0], w.wave, w.lane, 0);
    if constexpr (NCB > 0) {
#pragma unroll
        for (int rb = 0; rb < 4; ++rb)
            acc[rb][NCB - 1] = pend[rb] * ps[rb & 1] + acc[rb][NCB - 1];
    }
}

}  // namespace

template <bool DOWN>
__device__ __forceinline__ void kloop8_any(const Tile8 &t, const Wave8 &w, const Ring8 (&ring)[3],
                                           f32x4 (&acc)[4][4], int ncbw)
{
    if (w.wt == 0) {
        switch (ncbw) {
        case 0: kloop8<true, 0, DOWN>(t, w, ring, acc); break;
        case 1: kloop8<true, 1, DOWN>(t, w, ring, acc); break;
        case 2: kloop8<true, 2, DOWN>(t, w, ring, acc); break;
        case 3: kloop8<true, 3, DOWN>(t, w, ring, acc); break;
        default: kloop8<true, 4, DOWN>(t, w, ring, acc); break;
        }
    } else {
        switch (ncbw) {
        case 0: kloop8<false, 0, DOWN>(t, w, ring, acc); break;
        case 1: kloop8<false, 1, DOWN>(t, w, ring, acc); break;
        case 2: kloop8<false, 2, DOWN>(t, w, ring, acc); break;
        case 3: kloop8<false, 3, DOWN>(t, w, ring, acc); break;
        default: kloop8<false, 4, DOWN>(t, w, ring, acc); break;
        }
    }
}

__global__ __launch_bounds__(kThreads8, 1)
void k_ffn_fp8(FfnArgs)
{
    KernArgs args = kernel_args();
    __shared__ __attribute__((aligned(1024))) uint8_t lds_w0[kWBytes];
    __shared__ __attribute__((aligned(1024))) uint8_t lds_w1[kWBytes];
    __shared__ __attribute__((aligned(1024))) uint8_t lds_w2[kWBytes];
    // token rows and token scales share one object per stage: the compiler
    // tracks a limited number of direct-to-LDS targets when it decides which
    // LDS reads must wait for which loads, and six stay within it
    __shared__ __attribute__((aligned(1024))) uint8_t lds_x0[kXSBytes];
    __shared__ __attribute__((aligned(1024))) uint8_t lds_x1[kXSBytes];
    __shared__ __attribute__((aligned(1024))) uint8_t lds_x2[kXSBytes];
    __shared__ float hmax[4][kTokT];                   // SwiGLU: |h| maximum per wave and token
    __shared__ SchedLds sl;
    const Ring8 ring[3] = {{lds_w0, lds_x0, (float *)(lds_x0 + kXBytes)},
                           {lds_w1, lds_x1, (float *)(lds_x1 + kXBytes)},
                           {lds_w2, lds_x2, (float *)(lds_x2 + kXBytes)}};

    int tid = threadIdx.x;
    Worker<true, false> wk;
    if (tid == 192) {                     // the layer's weights, while begin() loads
        const void *W1 = args->p1.W, *W2 = args->p2.W;
        const float *S1 = args->p1.Ws, *S2 = args->p2.Ws;
        if (args->layer_id) {
            int ly = *args->layer_id;
            if (ly < 0 || ly >= args->n_layers) {
                if (blockIdx.x == 0 && args->sched.hdr[0] > 0) atomicOr(args->err, kErrBadLayer);
                ly = ly < 0 ? 0 : args->n_layers - 1;
            }
            W1 = args->layers[ly].w1;
            W2 = args->layers[ly].w2;
            S1 = args->layers[ly].s1;
            S2 = args->layers[ly].s2;
        }
        sl.w[0] = (uint64_t)W1;
        sl.w[1] = (uint64_t)W2;
        sl.ws[0] = (uint64_t)S1;
        sl.ws[1] = (uint64_t)S2;
    }
    if (!wk.begin(args->sched, sl, args->phases, args->tiles)) return;

    for (;;) {
        args = reload(args);
        if (!wk.next(args->sched, sl, args->phases, args->tiles, args->err)) break;
        args = reload(args);
        // nothing that a lane derives from its number is kept over the items
        asm volatile("" : "+v"(tid));
        Wave8 w;
        w.lane = tid & 63;
        w.wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        w.wf = w.wave & 3;
        w.wt = w.wave >> 2;
        const int lane = w.lane;
        // MFMA operand reads.  Weight fragment rb of this wave: feature block
        // 4 wf + rb, lane-contiguous halves.  Token block cb: lane l takes token
        // 64 wt + 16 cb + l % 16 and the 32 bytes [32 (l / 16), + 32) of its row.
        {
            const int r = w.wt * 64 + (lane & 15), swz = x_swizzle(r), c0 = 2 * (lane >> 4);
            w.w_rd = w.wf * 4 * 2048 + lane * 16;
            w.x_rd0 = r * kGrpB + ((c0 ^ swz) << 4);
            w.x_rd1 = r * kGrpB + (((c0 + 1) ^ swz) << 4);
            w.s_rd = r;
        }
        const bool down = wk.down;
        const RowTile rt = wk.row_tile(args->sched, sl);
        const bool sh = rt.group == args->shared_group;
        const int N = down ? args->p2.N : args->p1.N, K = down ? args->p2.K : args->p1.K;
        const void *Ar = down ? args->p2.A_routed : args->p1.A_routed;
        const void *Ash = down ? args->p2.A_shared : args->p1.A_shared;
        const float *Sr = down ? args->p2.As_routed : args->p1.As_routed;
        const float *Ssh = down ? args->p2.As_shared : args->p1.As_shared;
        const int rows_valid = rt.rows, row0 = rt.row0, nt = wk.nt;
        const int n0 = nt * kFeatT;
        // routed rows of an indexed A are gathered in the token fills: tile
        // row r is row A_index[row0 + r] / A_index_div of the whole A (its
        // scales are already gathered, indexed by the routed row)
        const int32_t *index = (!down && !sh) ? args->A_index : nullptr;
        const uint8_t *A = index ? (const uint8_t *)Ar : (const uint8_t *)(sh ? Ash : Ar) + (int64_t)row0 * K;
        const float *As = (sh ? Ssh : Sr) + row0;      // [K/128][ld]
        const uint8_t *B = uniform_ptr((const uint8_t *)sl.w[down ? 1 : 0]) + ((int64_t)rt.group * N + n0) * K;
        const float *Bsw = uniform_ptr((const float *)sl.ws[down ? 1 : 0]);
        Tile8 t;
        t.KT = K / kGrpB;
        t.s_ld = sh ? args->lds_shared : args->lds_routed;
        t.ncb = min(kFeatT, N - n0) / 16;
        t.cbstride = t.KT * 2048;
        t.rw = rsrc8(B, (int64_t)t.ncb * t.cbstride);
        t.rx = rsrc8(A, (index ? args->A_routed_rows : (int64_t)rows_valid) * K);
        t.rs = rsrc8(As, ((int64_t)(t.KT - 1) * t.s_ld + rows_valid) * 4);
        {
            // token fills: lane l covers row 16 w + 8 i + l / 8, physical chunk l % 8
            int src[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int r = min(w.wave * 16 + 8 * i + (lane >> 3), rows_valid - 1);
                src[i] = index ? index[row0 + r] / args->A_index_div : r;
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int r = w.wave * 16 + 8 * i + (lane >> 3);
                t.vx[i] = r < rows_valid ? src[i] * K + (((lane & 7) ^ x_swizzle(r)) << 4) : (int)0x80000000u;
            }
        }
        const float *sbp0, *sbp1;
        if (!down) {
            // [G][f/128][gate, up][K/128]: tile nt covers gate/up scale block nt
            const int f = N / 2;
            sbp0 = Bsw + ((int64_t)rt.group * (f / 128) + nt) * 2 * t.KT;
            sbp1 = sbp0 + t.KT;
        } else {
            // [G][N/128][K/128]: wave features n0 + 64 wf .. + 63
            const int nb = min(2 * nt + (w.wf >> 1), N / 128 - 1);
            sbp0 = sbp1 = Bsw + ((int64_t)rt.group * (N / 128) + nb) * t.KT;
        }
        t.sbp0 = (const cfloat *)(uintptr_t)sbp0;
        t.sbp1 = (const cfloat *)(uintptr_t)sbp1;

        f32x4 acc[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = (f32x4){};

        // 16-token blocks of this wave's 64 tokens that hold tokens of the group
        const int ncbw = __builtin_amdgcn_readfirstlane(
            min(4, max(0, rows_valid - w.wt * 64 + 15) / 16));
        if (down) kloop8_any<true>(t, w, ring, acc, ncbw);
        else kloop8_any<false>(t, w, ring, acc, ncbw);
        __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));   // vmcnt(0): the clamped look-ahead fills
        __syncthreads();                                     // ring idle in every wave
        wk.request();

        // Accumulator register i of block (rb, cb) holds feature
        // 16 rb + 4 (lane / 16) + i of the wave and token 16 cb + lane % 16.
        const int tok = w.wt * 64 + (lane & 15);        // + 16 cb
        const int fq = 4 * (lane >> 4);                 // + 16 rb + i
        if (!down) {
            // Gate and up rows interleave by 16: blocks rb = 2 p and 2 p + 1 are
            // gate and up of h channels 32 wf + 16 p + 4 (lane / 16) + i of the
            // tile's 128, so every wave forms its own h.  A token's scale needs
            // |h| over all 128 channels: each wave reduces its 32 (lanes
            // l, l ^ 16, l ^ 32, l ^ 48 hold the same token), and the four
            // waves of the same tokens meet in LDS.  The codes are staged in the
            // ring and leave as whole 128-byte lines, past this XCD's L2 (the
            // down items that read them run on other XCDs in the same launch).
            const int f = N / 2;
            f32x4 h[2][4];
            float am[4];
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) {
                float m = 0.0f;
#pragma unroll
                for (int pq = 0; pq < 2; ++pq)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float hv = silu_mul(acc[2 * pq][cb][i], acc[2 * pq + 1][cb][i]);
                        h[pq][cb][i] = hv;
                        m = fmaxf(m, fabsf(hv));
                    }
                m = fmaxf(m, __shfl_xor(m, 16));
                am[cb] = fmaxf(m, __shfl_xor(m, 32));
                if (lane < 16) hmax[w.wf][tok + 16 * cb] = am[cb];
            }
            __syncthreads();
            float *Hs = (sh ? args->p1.Cs_shared : args->p1.Cs_routed) + (int64_t)nt * t.s_ld + row0;
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) {
                const int tk = tok + 16 * cb;
                const float amax = fmaxf(fmaxf(hmax[0][tk], hmax[1][tk]), fmaxf(hmax[2][tk], hmax[3][tk]));
                const float sc = amax > 0.0f ? amax / 448.0f : 1.0f;   // the activation quantiser's scale
                const float inv = __builtin_amdgcn_rcpf(sc);
                uint8_t *dst = lds_w0 + tk * kHStride8 + w.wf * 32 + fq;
#pragma unroll
                for (int pq = 0; pq < 2; ++pq)
                    *(uint32_t *)(dst + 16 * pq) = e4m3_pack4(h[pq][cb][0] * inv, h[pq][cb][1] * inv,
                                                              h[pq][cb][2] * inv, h[pq][cb][3] * inv);
                if (w.wf == 0 && lane < 16 && tk < rows_valid)
                    __hip_atomic_store(&Hs[tk], sc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            __syncthreads();
            const auto rh = rsrc8((uint8_t *)(sh ? args->p1.C_shared : args->p1.C_routed) + (int64_t)row0 * f,
                                  (int64_t)rows_valid * f);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int r = i * 64 + (tid >> 3), c = tid & 7;       // 16 bytes of a row's 128
                const u32x4 v = *(const u32x4 *)(lds_w0 + r * kHStride8 + c * 16);
                __builtin_amdgcn_raw_buffer_store_b128(v, rh, r * f + nt * 128 + c * 16, 0, kAgentScope8);
            }
        } else {
            bf16 *C = (bf16 *)(sh ? args->p2.C_shared : args->p2.C_routed);
            const int fb = n0 + w.wf * 64 + fq;
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) {
                const int tk = tok + 16 * cb;
                if (tk < rows_valid) {
                    bf16 *dst = C + (int64_t)(row0 + tk) * N + fb;
#pragma unroll
                    for (int rb = 0; rb < 4; ++rb) {
                        if (fb + rb * 16 < N) {
                            typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
                            const bf16x4 v = {f2bf(acc[rb][cb][0]), f2bf(acc[rb][cb][1]),
                                              f2bf(acc[rb][cb][2]), f2bf(acc[rb][cb][3])};
                            *(bf16x4 *)(dst + rb * 16) = v;
                        }
                    }
                }
            }
        }
        args = reload(args);
        wk.done(args->sched, sl, args->phases, args->tiles);
    }
}

hipError_t launch_ffn_fp8(const FfnArgs &a, int grid, hipStream_t s)
{
    hipLaunchKernelGGL(k_ffn_fp8, dim3(grid), dim3(kThreads8), 0, s, a);
    return hipGetLastError();
}

}  // namespace moe
