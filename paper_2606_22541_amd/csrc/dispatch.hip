// Dispatch of one micro-batch: per-expert histogram, scan, stable counting-sort
// scatter and the gather of the fp8 token scales.
//
// The per-expert token counts are the metadata the paper's MoE devices receive
// with each batch, and the payload is grouped by expert (section 3.2.1,
// Table 2).  Here the stage derives them itself from the top-k ids.
//
// The order within an expert is ascending slot index s = t*k + j.  It is
// produced without any atomic deciding an order: each workgroup owns a
// contiguous chunk of slots, each wave a contiguous part of the chunk, and
// ranks inside a 64-slot step come from wave ballots, so the result is the
// stable counting sort, bit for bit.
#include "kernels.h"

namespace moe {

constexpr int kWaves = kDispatchThreads / 64;
constexpr int kPerWave = kDispatchChunk / kWaves;     // slots per wave
constexpr int kSteps = kPerWave / 64;                 // 64-slot steps per wave

// Exclusive prefix sum of one value per thread over the workgroup; *total
// receives the sum of all values.  Every thread of the workgroup must call it.
__device__ int block_excl_scan(int v, int32_t *wsum, int &total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    if (lane == 63) wsum[wave] = x;
    __syncthreads();
    int pre = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const int t = wsum[w];
        if (w < wave) pre += t;
        tot += t;
    }
    __syncthreads();
    total = tot;
    return pre + x - v;
}

// ---------------------------------------------------------------------------
// 1. Histogram over all experts, one row of counts per workgroup of
//    kDispatchChunk slots.  Loads use clamped indices so that each thread
//    issues all of its loads before the first use.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kDispatchThreads)
void k_hist(const int32_t *__restrict__ ids, int32_t n_slots, int32_t E,
            int32_t *__restrict__ blk_counts, int32_t *__restrict__ err)
{
    __shared__ int32_t h[kMaxExperts];
    for (int e = threadIdx.x; e < E; e += kDispatchThreads) h[e] = 0;
    const int64_t base = (int64_t)blockIdx.x * kDispatchChunk + threadIdx.x;
    constexpr int kPer = kDispatchChunk / kDispatchThreads;
    int v[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int64_t sl = base + (int64_t)j * kDispatchThreads;
        v[j] = ids[sl < n_slots ? sl : n_slots - 1];
    }
    __syncthreads();
    int bad = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        if (base + (int64_t)j * kDispatchThreads >= n_slots) continue;
        if (v[j] >= 0 && v[j] < E) atomicAdd(&h[v[j]], 1);   // integer counts: order-free
        else if (v[j] != -1) bad = 1;
    }
    if (bad) atomicOr(err, kErrBadId);
    __syncthreads();
    for (int x = threadIdx.x; x < E; x += kDispatchThreads)
        blk_counts[(int64_t)blockIdx.x * E + x] = h[x];
}

// Exclusive prefix sum over the 64 lanes of a wave; *total receives the sum.
__device__ __forceinline__ int wave_excl_scan(int v, int lane, int &total)
{
    int x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    total = __shfl(x, 63);
    return x - v;
}

__device__ __forceinline__ int wave_sum(int v)
{
#pragma unroll
    for (int o = 32; o; o >>= 1) v += __shfl_xor(v, o);
    return __builtin_amdgcn_readfirstlane(v);
}

// The row tiles of the FFN pass (ffn_sched.h) over G = E_loc (+1 shared)
// groups, built by one workgroup; a group's rows are the local expert's token
// count (tot), or T for the shared expert.
//
// A large group is split evenly into as few row tiles of at most h 32-row
// blocks as hold its rows.  h is the largest height, which does the most
// work per weight read, unless the gate/up product then leaves workgroups
// without an item: the pass would last as long as its largest tile, so h is
// the smallest for which the items still fit in one round (a small item
// counted as a third of a large one: it takes 50 to 80 us at d = 7168, against
// 150 to 200).  EP32 share at T = 8191, about 261 rows an expert: two tiles of
// 160 and 128 rows instead of one of 288, 301 -> 266 us a layer; 2300 pre-grouped
// rows of 8 uneven experts 294 -> 238.  T = 32768 has more items than workgroups either way.
// The first wave builds (in chunks of 64 groups, with shuffle scans and no
// workgroup barrier: the other workgroups place their slots meanwhile), the
// other waves clear the counters of the next pass.
__device__ void build_schedule(const Sched &s, const SchedPlan &plan, const int32_t *tot,
                               int E_loc, int has_shared, int T)
{
    const int G = E_loc + (has_shared ? 1 : 0);
    if (threadIdx.x >= 64) {
        for (int i = threadIdx.x - 64; i < kSchedTicks; i += kDispatchThreads - 64) s.tick[i] = 0;
        for (int i = threadIdx.x - 64; i < kMaxSchedCus; i += kDispatchThreads - 64) s.claim[i] = 0;
        return;
    }
    const int lane = threadIdx.x;
    auto rows_of = [&](int i) { return i < E_loc ? tot[i] : (i < G ? T : 0); };
    // the gate/up items with the largest tiles, and, if they leave workgroups
    // idle, the smallest height with which they still fit one round
    int n_small = 0, n10 = 0;
    bool any_large = false, tall = false, other = false;
    for (int c0 = 0; c0 < G; c0 += 64) {
        const int rows = rows_of(c0 + lane);
        n_small += __popcll(__ballot(rows > 0 && rows <= plan.small_rows));
        any_large |= __ballot(rows > plan.small_rows) != 0;
        tall |= __ballot(rows > 32 * plan.max_blocks) != 0;
        other |= __ballot(rows > 0 && rows <= plan.small_rows) != 0;
        n10 += rows > plan.small_rows ? (((rows + 31) >> 5) + plan.max_blocks - 1) / plan.max_blocks : 0;
    }
    const int room = plan.grid - n_small * plan.nt_small / 3;
    int h = plan.max_blocks;
    const int n_min = any_large ? wave_sum(n10) : 0;      // row tiles of the largest height
    if (any_large && plan.min_blocks < plan.max_blocks && n_min * plan.nt_large <= room) {
        // lane h: the items with tiles of h blocks (few groups: each makes one
        // row tile at least)
        const int hl = min(max(lane, plan.min_blocks), plan.max_blocks);
        int n = 0;
        for (int i = 0; i < G; ++i) {
            const int rows = rows_of(i);
            n += rows > plan.small_rows ? (((rows + 31) >> 5) + hl - 1) / hl : 0;
        }
        const uint64_t fits = __ballot(lane >= plan.min_blocks && lane <= plan.max_blocks && n * plan.nt_large <= room);
        h = __ffsll((unsigned long long)fits) - 1;
    }
    // row tiles of each class (large, small above plan.small_rows_down rows, small),
    // then every group's first row and first row tile
    auto tiles_of = [&](int rows) { return rows > plan.small_rows ? (((rows + 31) >> 5) + h - 1) / h : rows > 0 ? 1 : 0; };
    auto class_of = [&](int rows) { return rows > plan.small_rows ? 0 : rows > plan.small_rows_down ? 1 : 2; };
    int n_large = 0, n_mid = 0, n_all = 0;
    for (int c0 = 0; c0 < G; c0 += 64) {
        const int rows = rows_of(c0 + lane), m = tiles_of(rows);
        int t;
        wave_excl_scan(class_of(rows) == 0 ? m : 0, lane, t);
        n_large += t;
        n_mid += __popcll(__ballot(m > 0 && class_of(rows) == 1));
        n_all += t + __popcll(__ballot(m > 0 && class_of(rows) != 0));
    }
    // The down product's own row tiles.  Where the gate/up product splits its
    // groups to fill one round, the down product's items are more than one
    // round, and without the split they are one: it takes each group in one
    // tile then, and reads its weights once.  T = 8191: 92 -> 78 us for the
    // product, 276 -> 264 for the layer.  Only where every group is large and
    // none needs several tiles anyway: with hot groups among cold ones, of
    // which some down tiles were taller then, 2300 skewed rows took 258 us
    // instead of 243, four skewed micro-batches at once 1064 instead of 1053.
    const bool own = n_large > n_min && !tall && !other && n_large <= kSchedLdsTiles &&
                     n_large * plan.nt_down > plan.grid && n_min * plan.nt_down <= plan.grid;
    int c_group = 0;
    int c_row = 0, c_large = 0, c_mid = n_large, c_small = n_large + n_mid;
    int4 *rt = (int4 *)s.rt;
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    for (int c0 = 0; c0 < G; c0 += 64) {
        const int i = c0 + lane, rows = rows_of(i), m = tiles_of(rows), c = class_of(rows);
        int t_row, t_large;
        const int p_row = wave_excl_scan(i < E_loc ? rows : 0, lane, t_row);
        const int p_large = wave_excl_scan(c == 0 ? m : 0, lane, t_large);
        const uint64_t mid = __ballot(m > 0 && c == 1), small = __ballot(m > 0 && c == 2);
        const int row0 = i < E_loc ? c_row + p_row : 0;
        if (own) {
            const uint64_t some = __ballot(m > 0);
            const int at = c_group + __popcll(some & below);
            if (m > 0)
                rt[n_all + at] = make_int4(i | m << 16 | 1 << 30, row0, rows | 1 << 9 | (c_large + p_large) << 19, at);
            c_group += __popcll(some);
        }
        if (m > 0) {
            const int at = c == 0 ? c_large + p_large : c == 1 ? c_mid + __popcll(mid & below)
                                                               : c_small + __popcll(small & below);
            const int nb = (rows + 31) >> 5, q = nb / m, r = nb - q * m;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int first = 32 * (k * q + min(k, r));
                if (k < m)
                    rt[at + k] = make_int4(i | (m == 1 ? 1 << 30 : 0), row0 + first,
                                           min(32 * (q + (k < r ? 1 : 0)), rows - first) | m << 9, at);
            }
        }
        // the further row tiles of groups of more than four: the wave together
        for (uint64_t todo = __ballot(m > 4); todo; todo &= todo - 1) {
            const int v = __ffsll((unsigned long long)todo) - 1;
            const int vr = __builtin_amdgcn_readlane(rows, v), vm = __builtin_amdgcn_readlane(m, v);
            const int v0 = __builtin_amdgcn_readlane(row0, v);
            const int va = c_large + __builtin_amdgcn_readlane(p_large, v);
            const int nb = (vr + 31) >> 5, q = nb / vm, r = nb - q * vm;
            for (int k = 4 + lane; k < vm; k += 64) {
                const int first = 32 * (k * q + min(k, r));
                rt[va + k] = make_int4(c0 + v, v0 + first,
                                       min(32 * (q + (k < r ? 1 : 0)), vr - first) | vm << 9, va);
            }
        }
        c_row += t_row;
        c_large += t_large;
        c_mid += __popcll(mid);
        c_small += __popcll(small);
    }
    for (int i = lane; i < n_all; i += 64) s.dep[i * kDepStride] = 0;
    if (lane == 0) {
        s.hdr[0] = n_all;
        s.hdr[1] = n_large;
        s.hdr[2] = own ? n_min : n_large + n_mid;
        s.hdr[3] = own ? n_min : n_all;
        s.hdr[4] = own ? n_all : 0;
    }
}

// The counters of a schedule as the build leaves them, for a second pass over
// the same row tiles.
__global__ __launch_bounds__(kDispatchThreads)
void k_reset_schedule(Sched s)
{
    for (int i = threadIdx.x; i < kSchedTicks; i += kDispatchThreads) s.tick[i] = 0;
    for (int i = threadIdx.x; i < kMaxSchedCus; i += kDispatchThreads) s.claim[i] = 0;
    const int n = s.hdr[0];
    for (int i = threadIdx.x; i < n; i += kDispatchThreads) s.dep[i * kDepStride] = 0;
}

hipError_t launch_reset_schedule(const Sched &s, hipStream_t st)
{
    hipLaunchKernelGGL(k_reset_schedule, dim3(1), dim3(kDispatchThreads), 0, st, s);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// 2. Placement.  Workgroup b owns the same kDispatchChunk slots as histogram
//    workgroup b; wave w owns slots [b*chunk + w*chunk/4, b*chunk +
//    (w+1)*chunk/4) and walks them in 64-slot steps.  Every workgroup reads
//    the local-expert columns of the histogram rows to get the expert totals
//    and the counts of the workgroups before it, so no single-workgroup scan
//    sits between the two kernels.  Workgroup b also writes the global counts
//    of experts b, b + grid, ...; workgroup 0 writes the offsets, and the
//    last workgroup, which owns no slots, the FFN pass's row tiles.
//    Within a step, lanes holding the same expert are ranked by lane order
//    with a ballot.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kDispatchThreads)
void k_place(const int32_t *__restrict__ ids, int32_t n_slots, int32_t nb_hist, int32_t E,
             int32_t e0, int32_t E_loc, int32_t T, int32_t has_shared,
             const int32_t *__restrict__ blk_counts, int32_t *__restrict__ counts,
             int32_t *__restrict__ offsets, Sched sched, SchedPlan plan,
             int32_t *__restrict__ slot_of_row, int32_t *__restrict__ row_of_slot)
{
    __shared__ int32_t tot[kMaxLocalExperts], pre[kMaxLocalExperts];
    __shared__ int32_t wbase[kWaves][kMaxLocalExperts];
    __shared__ int32_t cnt_my[kMaxExperts];
    __shared__ int32_t wsum[kWaves];
    const int b = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int64_t wstart = (int64_t)b * kDispatchChunk + (int64_t)wave * kPerWave + lane;

    // The ids loads are issued first; the LDS set-up uses a barrier that
    // waits for LDS stores only, so the histogram-row loads below are
    // issued while the ids are still in flight (one latency, not two).
    int v[kSteps];
    if (n_slots > 0) {
#pragma unroll
        for (int j = 0; j < kSteps; ++j) {
            const int64_t sl = wstart + j * 64;
            v[j] = ids[sl < n_slots ? sl : n_slots - 1];
        }
    }
    const int n_my = b < E ? (E - 1 - b) / (int)gridDim.x + 1 : 0;
    for (int i = tid; i < E_loc; i += kDispatchThreads) {
        tot[i] = 0;
        pre[i] = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) wbase[w][i] = 0;
    }
    for (int q = tid; q < n_my; q += kDispatchThreads) cnt_my[q] = 0;
    // first histogram value of this thread's share of the global counts,
    // loaded now so that it arrives with the ones below instead of a round
    // trip later
    const int n_cnt = n_my * nb_hist;
    int cnt0 = 0;
    if (tid < n_cnt) {
        const int q = tid / nb_hist, bb = tid - q * nb_hist;
        cnt0 = blk_counts[(int64_t)bb * E + b + q * (int)gridDim.x];
    }
    __builtin_amdgcn_s_waitcnt((15) | (3 << 14) | (7 << 4) | (0 << 8));   // lgkmcnt(0) only
    __builtin_amdgcn_s_barrier();

    // expert totals and the part of them in earlier workgroups
    {
        const int tpe = E_loc < kDispatchThreads ? kDispatchThreads / E_loc : 1;
        const int i = tid / tpe, sub = tid - i * tpe;
        if (i < E_loc) {
            // eight loads in flight: a thread's rows are tpe apart
            int t = 0, p = 0, bb = sub;
            for (; bb + 3 * tpe < nb_hist; bb += 8 * tpe) {
                int c[8];
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    c[u] = blk_counts[(int64_t)min(bb + u * tpe, nb_hist - 1) * E + e0 + i];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int r = bb + u * tpe;
                    t += r < nb_hist ? c[u] : 0;
                    p += r < min(nb_hist, b) ? c[u] : 0;
                }
            }
            for (; bb < nb_hist; bb += tpe) {
                const int c = blk_counts[(int64_t)bb * E + e0 + i];
                t += c;
                p += bb < b ? c : 0;
            }
            atomicAdd(&tot[i], t);
            atomicAdd(&pre[i], p);
        }
    }
    // local expert index of each slot this lane owns (-1: not local / none)
    int li[kSteps];
#pragma unroll
    for (int j = 0; j < kSteps; ++j) {
        const int i = v[j] - e0;
        li[j] = (n_slots > 0 && wstart + j * 64 < n_slots && v[j] >= 0 && v[j] < E && i >= 0 &&
                 i < E_loc) ? i : -1;
    }
    // per-wave counts of this workgroup's slots
#pragma unroll
    for (int j = 0; j < kSteps; ++j)
        if (li[j] >= 0) atomicAdd(&wbase[wave][li[j]], 1);
    // global counts of experts b, b + grid, ...
    if (tid < n_cnt) atomicAdd(&cnt_my[tid / nb_hist], cnt0);
    for (int it = tid + kDispatchThreads; it < n_cnt; it += kDispatchThreads) {
        const int q = it / nb_hist, bb = it - q * nb_hist;
        atomicAdd(&cnt_my[q], blk_counts[(int64_t)bb * E + b + q * (int)gridDim.x]);
    }
    __syncthreads();
    for (int q = tid; q < n_my; q += kDispatchThreads) counts[b + q * (int)gridDim.x] = cnt_my[q];

    // the last workgroup owns no slots (the launch adds it for this): it
    // builds the FFN's row tiles while the others place their slots
    if (b == (int)gridDim.x - 1 && b > 0) {
        if (sched.hdr) build_schedule(sched, plan, tot, E_loc, has_shared, T);
        return;
    }

    // offsets (E_loc <= 256: one local expert per thread) and wave bases
    int total = 0;
    const int off_i = block_excl_scan(tid < E_loc ? tot[tid] : 0, wsum, total);
    if (tid < E_loc) {
        int run = off_i + pre[tid];
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const int t = wbase[w][tid];
            wbase[w][tid] = run;
            run += t;
        }
    }
    if (b == 0) {
        if (tid < E_loc) offsets[tid] = off_i;
        if (tid == 0) offsets[E_loc] = total;
    }
    __syncthreads();

    // Lanes of a step that hold the same expert find each other by one ballot
    // for each bit of the local index (a loop over the step's distinct experts
    // took a round trip through LDS for each of them), and rank by lane order.
    volatile int32_t *mybase = wbase[wave];
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int bits = 32 - __clz(E_loc - 1 | 1);
#pragma unroll
    for (int j = 0; j < kSteps; ++j) {
        const int64_t sl = wstart + j * 64;
        const int i = li[j];
        uint64_t peers = __ballot(i >= 0);
        for (int t = 0; t < bits; ++t) {
            const bool one = i >> t & 1;
            const uint64_t m = __ballot(one);
            peers &= one ? m : ~m;
        }
        int pos = -1;
        if (i >= 0) {
            const int bse = mybase[i];
            const int rank = __popcll(peers & lt_mask);
            pos = bse + rank;
            if (rank == 0) mybase[i] = bse + __popcll(peers);
        }
        if (sl < n_slots) {
            row_of_slot[sl] = pos;
            if (pos >= 0) slot_of_row[pos] = (int32_t)sl;
        }
    }
    // without slots there is one workgroup only
    if (gridDim.x == 1 && sched.hdr) build_schedule(sched, plan, tot, E_loc, has_shared, T);
}

// Row tiles for pre-grouped rows (the receive region of section 3.2.1 in
// its grouped form: the senders supply the per-expert counts).  One
// workgroup: its first wave validates the counts in order, then the same
// build as the dispatch.
__global__ __launch_bounds__(kDispatchThreads)
void k_group_tables_from_counts(const int32_t *__restrict__ counts, int32_t E_loc,
                                int32_t n_rows_max, Sched sched, SchedPlan plan,
                                int32_t *__restrict__ err)
{
    __shared__ int32_t tot[kMaxLocalExperts];
    const int lane = threadIdx.x;
    if (lane < 64) {
        int carry = 0, bad = 0;
        for (int c0 = 0; c0 < E_loc; c0 += 64) {
            const int i = c0 + lane;
            const int c = i < E_loc ? counts[i] : 0, asked = rows_asked(c, n_rows_max);
            // sums capped at n_rows_max, so that no counts can wrap them
            int x = asked;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_up(x, o);
                if (lane >= o) x = add_capped(x, y, n_rows_max);
            }
            const int y = __shfl_up(x, 1);
            const int before = add_capped(carry, lane ? y : 0, n_rows_max);
            // rows past n_rows_max are dropped: the group keeps what fits
            const int keep = rows_kept(asked, before, n_rows_max);
            bad |= keep != c;
            if (i < E_loc) tot[i] = keep;
            carry = add_capped(carry, __shfl(x, 63), n_rows_max);
        }
        if (__any(bad) && lane == 0) atomicOr(err, kErrBadCount);
    }
    __syncthreads();
    build_schedule(sched, plan, tot, E_loc, 0, 0);
}

hipError_t launch_group_tables_from_counts(const int32_t *counts, int32_t E_loc,
                                           int32_t n_rows_max, const Sched &sched,
                                           const SchedPlan &plan, int32_t *err, hipStream_t s)
{
    hipLaunchKernelGGL(k_group_tables_from_counts, dim3(1), dim3(kDispatchThreads), 0, s, counts, E_loc,
                       n_rows_max, sched, plan, err);
    return hipGetLastError();
}

hipError_t launch_dispatch_index(const DispatchArgs &a, hipStream_t s)
{
    const int nb = (a.n_slots + kDispatchChunk - 1) / kDispatchChunk;
    if (nb > 0) {
        hipLaunchKernelGGL(k_hist, dim3(nb), dim3(kDispatchThreads), 0, s, a.ids, a.n_slots, a.E,
                           a.blk_counts, a.err);
    }
    // one workgroup per histogram row, plus one without slots for the row tiles
    hipLaunchKernelGGL(k_place, dim3(nb + 1), dim3(kDispatchThreads), 0, s, a.ids,
                       a.n_slots, nb, a.E, a.e0, a.E_loc, a.T, a.has_shared, a.blk_counts,
                       a.counts, a.offsets, a.sched, a.plan, a.slot_of_row, a.row_of_slot);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// 4. Scale gather (fp8): the grouped GEMMs read the token rows of x through
//    slot_of_row themselves, but they take the step's token scales as one
//    contiguous run per 128-channel group, so the scales of the routed rows
//    are gathered here into the transposed [n_scales][scale_ld] layout.
//    Work item i (grid-stride) moves the scales of groups 8 (i / n_rows) ..
//    + 7 of row i % n_rows: the stores of a group are consecutive across a
//    wave, and each thread has its eight loads in flight at once.
// ---------------------------------------------------------------------------
constexpr int kGatherThreads = 256;
constexpr int kScalesPerItem = 8;

__global__ __launch_bounds__(kGatherThreads)
void k_gather_scales(const float *__restrict__ xs, const int32_t *__restrict__ slot_of_row,
                     const int32_t *__restrict__ n_rows_dev, int32_t k, int32_t n_scales,
                     float *__restrict__ xps, int32_t scale_ld)
{
    const int n_rows = *n_rows_dev;
    if (n_rows <= 0) return;
    const int64_t chunks = (n_scales + kScalesPerItem - 1) / kScalesPerItem;
    const int64_t total = (int64_t)n_rows * chunks;
    for (int64_t i = (int64_t)blockIdx.x * kGatherThreads + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * kGatherThreads) {
        const int c = (int)(i / n_rows);
        const int r = (int)(i - (int64_t)c * n_rows);
        const int g0 = c * kScalesPerItem;
        const float *src = xs + (int64_t)(slot_of_row[r] / k) * n_scales;
        float v[kScalesPerItem];
#pragma unroll
        for (int u = 0; u < kScalesPerItem; ++u) v[u] = src[min(g0 + u, n_scales - 1)];
#pragma unroll
        for (int u = 0; u < kScalesPerItem; ++u)
            if (g0 + u < n_scales) xps[(int64_t)(g0 + u) * scale_ld + r] = v[u];
    }
}

hipError_t launch_gather_scales(const float *x_scales, const int32_t *slot_of_row,
                                const int32_t *n_rows_dev, int32_t k, int32_t n_scales,
                                float *x_perm_scales, int32_t scale_ld, int32_t max_rows,
                                int num_cus, hipStream_t s)
{
    if (max_rows <= 0 || n_scales <= 0) return hipSuccess;
    const int64_t work = (int64_t)max_rows * ((n_scales + kScalesPerItem - 1) / kScalesPerItem);
    int64_t grid = (work + kGatherThreads - 1) / kGatherThreads;
    if (grid > (int64_t)num_cus * 4) grid = (int64_t)num_cus * 4;
    hipLaunchKernelGGL(k_gather_scales, dim3((unsigned)grid), dim3(kGatherThreads), 0, s, x_scales,
                       slot_of_row, n_rows_dev, k, n_scales, x_perm_scales, scale_ld);
    return hipGetLastError();
}

__global__ void k_transpose_scales(const float *__restrict__ src, int32_t rows, int32_t cols,
                                   float *__restrict__ dst, int32_t ld)
{
    const int64_t total = (int64_t)rows * cols;
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < total;
         q += (int64_t)gridDim.x * blockDim.x) {
        const int r = (int)(q / cols);
        const int c = (int)(q - (int64_t)r * cols);
        dst[(int64_t)c * ld + r] = src[q];
    }
}

hipError_t launch_transpose_scales(const float *src, int32_t rows, int32_t cols, float *dst,
                                   int32_t ld, hipStream_t s)
{
    const int64_t total = (int64_t)rows * cols;
    if (total <= 0) return hipSuccess;
    int64_t grid = (total + 255) / 256;
    if (grid > 1024) grid = 1024;
    hipLaunchKernelGGL(k_transpose_scales, dim3((unsigned)grid), dim3(256), 0, s, src, rows, cols,
                       dst, ld);
    return hipGetLastError();
}

}  // namespace moe
