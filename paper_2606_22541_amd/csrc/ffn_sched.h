// Device-side schedule of the expert FFN's persistent kernels: the row tiles
// of a pass, built by the dispatch, and the work lists that the workgroups of
// one launch take items from.
//
// Row tiles (int4 {group | only << 30, row0, rows | m << 9, first}: the group
// has m row tiles from `first` on): the large groups' tiles, group by group,
// then the small groups'.  Where the down product does not split the groups that
// the gate/up product splits, its row tiles, one a group and all of them large,
// follow as a table of their own ({group | m of gate/up << 16 | 1 << 30, row0,
// rows | 1 << 9 | first of gate/up << 19, first}), and the written gate/up tiles
// are counted per group (at the group's first row tile) instead of per row tile.
// An item of a product is (row tile, column tile); items are numbered group
// by group, within a large group in bands of a few row tiles (row tiles
// fastest, so that one band's weight panels and token rows are shared in an
// L2).
//
// Lists.  Workgroups are placed round-robin on the 8 XCDs, so the items of a
// product are dealt to 8 lists in runs of P / 8 consecutive items (P = the
// grid), one list per XCD: the workgroups of an XCD take them in order.  Fewer
// items than workgroups are dealt evenly all the same, so that the weights come
// through every XCD (deal.h).  The first run of a list's gate/up items is fixed,
// one per workgroup (no ticket has to come back before the first loads); later
// items are taken with an atomic ticket per list, requested while the previous
// item runs.  A workgroup whose list is empty takes from the others'.
//
// A down item waits until every gate/up tile of its rows is written (a count
// per row tile, each on a line of its own: polled on a shared line the waits
// of one product slowed the weights' stream of the other, 178 against 171 us at
// T = 4096).  Waiting cannot deadlock, whatever else runs on the GPU and
// however few workgroups are resident: a workgroup takes a down item only
// after its own list's gate/up items are taken, and one that has to wait
// looks for gate/up items that nobody has taken (in other lists, or fixed to
// workgroups that have not started) and runs those first.  So every gate/up
// item not yet finished is being run by a resident workgroup, which never
// waits.
#pragma once

#include "common.h"
#include "deal.h"

namespace moe {

constexpr int kMaxSchedCus = 512;     // workgroups of one launch
constexpr int kTickStride = 32;       // ints between ticket counters (128 bytes)
constexpr int kDepStride = 32;        // ints between row tiles' counts of written tiles
// Polls of one wait before it gives up (seconds; a wait takes microseconds).
constexpr int kMaxPolls = 1 << 22;
constexpr int kMaxReadyScan = 1024;   // row tiles that one wait looks over for "all are ready"

struct Sched {
    int32_t *rt;       // [n] int4 row tiles
    // row tiles, large ones of gate/up, large ones of down; row tiles of the
    // down product, where its table begins (0: the same table)
    int32_t *hdr;
    int32_t *dep;      // [n] gate/up tiles written, per row tile, kDepStride apart
    int32_t *claim;    // [kMaxSchedCus] fixed first item taken, per workgroup
    int32_t *tick;     // [2][kLists] tickets, kTickStride apart
};

// The schedule as a kernel argument, in the kernel-argument segment.
typedef const __attribute__((address_space(4))) Sched ArgSched;

constexpr int kSchedHdr = 64;
constexpr int kSchedHdrInts = 5;
constexpr int kSchedTicks = 2 * kLists * kTickStride;

// Row tiles that G groups with `rows` rows in all can make.
__host__ __device__ inline int64_t sched_max_tiles(int64_t rows, int64_t G)
{
    return rows / 128 + 2 * (G + kMaxSchedCus);
}
// Ints of a schedule, and its arrays in one allocation.
inline int64_t sched_ints(int64_t max_tiles)
{
    return kSchedHdr + kSchedTicks + kMaxSchedCus + (4 + kDepStride) * max_tiles;
}
inline Sched sched_at(int32_t *base, int64_t max_tiles)
{
    Sched s;
    s.hdr = base;
    s.tick = base + kSchedHdr;
    s.claim = s.tick + kSchedTicks;
    s.rt = s.claim + kMaxSchedCus;
    s.dep = s.rt + 4 * max_tiles;
    return s;
}

struct RowTile {
    int group, row0, rows;
    bool only;         // the group's only row tile
};

// What a workgroup keeps of the schedule in LDS (its registers belong to the
// tiles' loops).
constexpr int kSchedLdsTiles = 64;
struct SchedLds {
    int4 rt[kSchedLdsTiles];
    int32_t hdr[kSchedHdrInts];
    int32_t claimed, wait;     // begin(): the fixed item was taken; next(): what the wait found
    int32_t item, rti, nt;     // the next item and its tile (bit 30 of rti: a large one)
    int32_t ahead;             // done(): the next item is known
    int32_t run[2];            // run lengths of the two products' items
    int32_t stage;     // thread 0: list being drained (0 gate/up, 1 down, 2 the others')
    uint64_t w[2], ws[2];   // weights of the two products, and their scales
};

// The thread's number, as a value that the compiler does not keep (nor what
// it derives from it) in registers from one item to the next.
__device__ __forceinline__ int fresh_tid()
{
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

__device__ __forceinline__ int agent_load(const int32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int agent_add(int32_t *p, int v)
{
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int agent_swap(int32_t *p, int v)
{
    return __hip_atomic_exchange(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Column tiles of the two products, in the kernel's arguments.
struct FfnTiles {
    int32_t ntl[2];    // of a large row tile (256 columns)
    int32_t nts[2];    // of a small row tile (128 columns)
    int32_t band;      // row tiles of a raster band
    int32_t row_bytes; // of an activation row
};

typedef const __attribute__((address_space(4))) FfnTiles ArgTiles;

// The items of a launch and how they are dealt to lists.
struct Items : Deal {
    int x;                     // this workgroup's list
    int nrt, nl0, nl1;         // row tiles, large ones of gate/up and of down
    int nrtd, sd;              // row tiles of down, the start of their table
    int ntl0, ntl1, nts0, nts1, band;

    // FIRST: the run lengths are computed; otherwise they are in LDS.
    template <bool LARGE, bool OWN, bool FIRST = false>
    __device__ __forceinline__ void load(const SchedLds &l, int phases, ArgTiles &ct)
    {
        nrt = __builtin_amdgcn_readfirstlane(l.hdr[0]);
        nl0 = LARGE ? __builtin_amdgcn_readfirstlane(l.hdr[1]) : 0;
        nl1 = LARGE ? __builtin_amdgcn_readfirstlane(l.hdr[2]) : 0;
        nrtd = OWN ? __builtin_amdgcn_readfirstlane(l.hdr[3]) : nrt;
        sd = OWN ? __builtin_amdgcn_readfirstlane(l.hdr[4]) : 0;
        ntl0 = ct.ntl[0];
        ntl1 = ct.ntl[1];
        nts0 = ct.nts[0];
        nts1 = ct.nts[1];
        band = ct.band;
        const int g = nl0 * ntl0 + (nrt - nl0) * nts0, d = nl1 * ntl1 + (nrtd - nl1) * nts1;
        count(gridDim.x, g, d, phases);
        if constexpr (FIRST) deal(gridDim.x, g, d, ct.row_bytes);
        C = __builtin_amdgcn_readfirstlane(FIRST ? C : l.run[0]);
        C1 = __builtin_amdgcn_readfirstlane(FIRST ? C1 : l.run[1]);
        x = blockIdx.x & ((1 << lg) - 1);
    }
    // gate/up tiles that the count of gate/up row tile rt comes to
    __device__ __forceinline__ int need(int rt) const { return rt < nl0 ? ntl0 : nts0; }
};

// One workgroup's place in the lists.
// LARGE: large tiles occur.  OWN: the down product may have row tiles of its own.
template <bool LARGE, bool OWN = LARGE>
struct Worker {
    int pending;                 // a down item put off for a gate/up item, or -1
    int first;                   // the fixed first item, or -1
    bool have;                   // done() may have taken the next item (l.ahead)
    bool all_done;               // every row tile's gate/up tiles are written
    // current item
    bool down, large;
    int rti, nt;
    int32_t *next_tick;          // counter of the next ticket, or null
    int pre;                     // thread 0: requested ticket, or -1

    __device__ __forceinline__ bool begin(ArgSched &s, SchedLds &l, int phases, ArgTiles &ct)
    {
        const int tid = threadIdx.x, b = blockIdx.x;
        if (tid < kSchedLdsTiles) l.rt[tid] = ((const int4 *)s.rt)[tid];
        else if (tid < kSchedLdsTiles + kSchedHdrInts) l.hdr[tid - kSchedLdsTiles] = s.hdr[tid - kSchedLdsTiles];
        else if (tid == 128) l.claimed = (phases & 1) ? agent_swap(&s.claim[b], 1) : 1;
        __syncthreads();
        Items q;
        q.load<LARGE, OWN, true>(l, phases, ct);
        l.run[0] = q.C;          // (every wave the same, and each reads its own)
        l.run[1] = q.C1;
        all_done = false;
        pending = -1;
        pre = -1;
        const int run = q.C << q.lg;
        first = q.fixed(b);
        if (__builtin_amdgcn_readfirstlane(l.claimed) != 0) first = -1;
        have = false;
        if (tid == 0) l.stage = run + q.x * q.C < q.total0 ? 0 : 1;   // a second run of this list
        return q.total0 + q.total1 > 0;
    }

    static __device__ __forceinline__ int32_t *tick_of(ArgSched &s, int p, int y)
    {
        return s.tick + (p * kLists + y) * kTickStride;
    }

    __device__ __forceinline__ static int4 entry(ArgSched &s, const SchedLds &l, int rt)
    {
        int4 v;
        if (rt < kSchedLdsTiles) v = l.rt[rt];
        else v = ((const int4 *)s.rt)[rt];
        return v;
    }

    // The count that the down items of row tile rt (its place in the table)
    // wait for, and what it comes to.
    static __device__ __forceinline__ const int32_t *dep_of(ArgSched &s, const SchedLds &l, const Items &q, int rt,
                                                            int &need)
    {
        int c = rt;
        need = 1;
        if (OWN && q.sd) {
            const int4 e = entry(s, l, rt);
            c = e.z >> 19;
            need = e.x >> 16 & 0x3fff;
        }
        need *= q.need(c);
        return &s.dep[c * kDepStride];
    }

    // A ticket of product p, list y (wave 0; every lane gets it).
    static __device__ __forceinline__ int ticket(ArgSched &s, int p, int y)
    {
        int j = 0;
        if ((fresh_tid() & 63) == 0) j = agent_add(tick_of(s, p, y), 1);
        return __builtin_amdgcn_readfirstlane(j);
    }
    // An item of another list, product in bit 30, or -1 (wave 0): lane
    // kLists p + y looks at list y of product p.  Items that can run at once
    // (gate/up items, and down items whose rows are ready) come first.
    static __device__ __forceinline__ int steal(ArgSched &s, const SchedLds &l, const Items &q)
    {
        const int lane = fresh_tid() & 63, p = lane >> kListsLog2 & 1, y = lane & (kLists - 1);
        const int first = p ? 0 : q.C;
        const int n = lane < 2 * kLists && y < 1 << q.lg ? q.len(p, y) : 0;
        for (;;) {
            const int j = n > 0 ? first + agent_load(tick_of(s, p, y)) : 0;
            const bool open = j < n;
            const uint64_t any = __ballot(open);
            if (!any) return -1;
            bool ready = open;
            if (open && p) {
                int rt, nt, need;
                find(s, l, q, q.item(j, y, 1), 1, rt, nt);
                const int32_t *dep = dep_of(s, l, q, rt, need);
                ready = agent_load(dep) >= need;
            }
            const uint64_t now = __ballot(ready);
            const int v = __ffsll((unsigned long long)(now ? now : any)) - 1;
            const int pp = v >> kListsLog2, yy = v & (kLists - 1);
            const int t = ticket(s, pp, yy) + (pp ? 0 : q.C);
            if (t < q.len(pp, yy)) return q.item(t, yy, pp) | pp << 30;
        }
    }
    // The item of the requested ticket, or -1: none was requested, or the list
    // is drained (wave 0).
    __device__ __forceinline__ int take_requested(SchedLds &l, const Items &q)
    {
        const int want = __builtin_amdgcn_readfirstlane(pre), stage = __builtin_amdgcn_readfirstlane(l.stage);
        pre = -1;
        if (want < 0 || stage > 1) return -1;
        const int j = stage ? want : q.C + want;
        if (j < q.len(stage, q.x)) return q.item(j, q.x, stage) | stage << 30;
        l.stage = stage + 1;
        return -1;
    }
    // Next item (wave 0).
    __device__ __forceinline__ int take(ArgSched &s, SchedLds &l, const Items &q)
    {
        int it = take_requested(l, q);
        while (it < 0) {
            const int stage = __builtin_amdgcn_readfirstlane(l.stage);
            if (stage > 1) return steal(s, l, q);
            pre = q.len(stage, q.x) > 0 ? ticket(s, stage, q.x) : 0;   // (any ticket is past an empty list)
            it = take_requested(l, q);
        }
        return it;
    }

    // Wave 0: puts the next item and its tile where every wave finds them.
    __device__ __forceinline__ void set_next(ArgSched &s, SchedLds &l, const Items &q, int it)
    {
        if (it >= 0) {
            int rt, n;
            const bool lg = find(s, l, q, it & ~(1 << 30), it >> 30, rt, n);
            l.rti = rt | (lg ? 1 << 30 : 0);
            l.nt = n;
        }
        l.item = it;
    }

    // Wave 0: waits until the rows of row tile rt are ready.  -1: they are,
    // -2: the rows of every row tile are, >= 0: a gate/up item to run first.
    static __device__ __forceinline__ int wait_or_help(ArgSched &s, const SchedLds &l, const Items &q, int rt,
                                                       int32_t *err)
    {
        const int lane = fresh_tid() & 63, nx = 1 << q.lg;
        int need;
        const int32_t *dep = dep_of(s, l, q, rt, need);
        // every gate/up item is taken (and stays so): looking for others costs a
        // poll five round trips to memory, so it ends once it finds none
        bool taken = false;
        for (int polls = 0;; ++polls) {
            // one load of one line a poll: many workgroups may be waiting, and
            // their polls share HBM channels with the others' streams
            if (__builtin_amdgcn_readfirstlane(agent_load(dep)) >= __builtin_amdgcn_readfirstlane(need)) {
                // with every row tile ready the workgroup's later items need
                // no poll (fp8, 270 row tiles: 1721 -> 1698 us a pass)
                bool mine = q.nrtd <= kMaxReadyScan;
                for (int i = lane; i < q.nrtd && i < kMaxReadyScan; i += 64) {
                    int n;
                    const int32_t *di = dep_of(s, l, q, q.sd + i, n);
                    mine &= agent_load(di) >= n;
                }
                return __all(mine) ? -2 : -1;
            }
            if (polls > 2 && !taken) {
                // gate/up items that no workgroup has taken: tickets ...
                const int y = lane & (kLists - 1);
                const bool open = lane < nx && q.C + agent_load(tick_of(s, 0, y)) < q.len(0, y);
                const uint64_t m = __ballot(open);
                if (m) {
                    const int yy = __ffsll((unsigned long long)m) - 1;
                    const int j = q.C + ticket(s, 0, yy);
                    if (j < q.len(0, yy)) return q.item(j, yy, 0);
                    continue;
                }
                // ... and the fixed ones of workgroups that have not started
                bool none = true;
                for (int b0 = 0; b0 < (int)gridDim.x; b0 += 64) {
                    const int b = b0 + lane;
                    const bool idle = b < (int)gridDim.x && q.fixed(b) >= 0 &&
                                      agent_load(&s.claim[min(b, (int)gridDim.x - 1)]) == 0;
                    const uint64_t c = __ballot(idle);
                    if (c) {
                        const int bb = b0 + __ffsll((unsigned long long)c) - 1;
                        int old = 0;
                        if (lane == 0) old = agent_swap(&s.claim[bb], 1);
                        old = __builtin_amdgcn_readfirstlane(old);
                        if (old == 0) return q.fixed(bb);
                        none = false;
                    }
                }
                taken = none;
            }
            if (polls >= kMaxPolls) {
                if (lane == 0) atomicOr(err, kErrStalled);
                return -1;
            }
            __builtin_amdgcn_s_sleep(8);
        }
    }

    // Row tile and column tile of item `it` of product p (any lane's own).
    static __device__ __forceinline__ bool find(ArgSched &s, const SchedLds &l, const Items &q, int it, int p,
                                                int &rt, int &nt)
    {
        const int nl = p ? q.nl1 : q.nl0, wl = p ? q.ntl1 : q.ntl0, ws = p ? q.nts1 : q.nts0;
        const bool large = it < nl * wl;
        const int base = OWN && p ? q.sd : 0;
        if (large) {
            // the items of a group's m row tiles from the first on, in bands
            const int r0 = it / wl;
            const int4 e = entry(s, l, base + r0);
            const int rt0 = e.w, m = e.z >> 9 & (base ? 0x3ff : -1);
            const int i = it - rt0 * wl;
            if (m <= q.band) {
                nt = i / m;
                rt = rt0 + i - nt * m;
            } else {
                const int b = i / (q.band * wl), r = i - b * q.band * wl;
                const int bm = min(q.band, m - b * q.band);
                nt = r / bm;
                rt = rt0 + b * q.band + r - nt * bm;
            }
        } else {
            const int i = it - nl * wl;
            const int j = i / ws;
            rt = nl + j;
            nt = i - j * ws;
        }
        rt += base;
        return large;
    }
    __device__ __forceinline__ void decode(ArgSched &s, const SchedLds &l, const Items &q, int it, int p)
    {
        int rt, n;
        large = __builtin_amdgcn_readfirstlane((int)find(s, l, q, it, p, rt, n)) != 0;
        rti = __builtin_amdgcn_readfirstlane(rt);
        nt = __builtin_amdgcn_readfirstlane(n);
    }

    // The workgroup's next item; false: none is left.
    __device__ __forceinline__ bool next(ArgSched &s, SchedLds &l, int phases, ArgTiles &ct, int32_t *err)
    {
        Items q;
        q.load<LARGE, OWN>(l, phases, ct);
        int it = pending, p;
        if (first >= 0 || it >= 0) {
            if (first >= 0) it = first;
            first = -1;
            pending = -1;
            p = it >> 30;
            it &= ~(1 << 30);
            decode(s, l, q, it, p);
        } else {
            if (!have || __builtin_amdgcn_readfirstlane(l.ahead) == 0) {
                if (fresh_tid() < 64) set_next(s, l, q, take(s, l, q));
                __syncthreads();
            }
            it = __builtin_amdgcn_readfirstlane(l.item);
            if (it < 0) return false;
            p = it >> 30;
            it &= ~(1 << 30);
            const int r = __builtin_amdgcn_readfirstlane(l.rti);
            rti = r & ~(1 << 30);
            large = r >> 30;
            nt = __builtin_amdgcn_readfirstlane(l.nt);
        }
        have = false;
        down = p != 0;
        if (p && phases == 3 && !all_done) {
            if (fresh_tid() < 64) {
                const int r = wait_or_help(s, l, q, rti, err);
                if (fresh_tid() == 0) l.wait = r;
            }
            __syncthreads();
            const int r = __builtin_amdgcn_readfirstlane(l.wait);
            if (r == -2) all_done = true;
            if (r >= 0) {
                pending = it | 1 << 30;
                down = false;
                decode(s, l, q, r, 0);
            }
        }
        // where the next ticket comes from (see request())
        const int stage = __builtin_amdgcn_readfirstlane(l.stage);
        next_tick = nullptr;
        if (pending < 0 && stage < 2 && (stage == 0 || q.total1 > 0)) next_tick = tick_of(s, stage, q.x);
        return true;
    }

    // Requests the next ticket: before an item's epilogue, so that it comes
    // back meanwhile.  Not earlier: an item that is taken long before it can
    // run keeps the workgroups that wait for it waiting.
    __device__ __forceinline__ void request()
    {
        if (next_tick && fresh_tid() == 0 && pre < 0) pre = agent_add(next_tick, 1);
    }

    __device__ __forceinline__ RowTile row_tile(ArgSched &s, const SchedLds &l) const
    {
        const int4 v = entry(s, l, rti);
        RowTile r;
        const int g = __builtin_amdgcn_readfirstlane(v.x);
        r.group = g & 0xffff;
        r.only = g >> 30;
        r.row0 = __builtin_amdgcn_readfirstlane(v.y);
        r.rows = __builtin_amdgcn_readfirstlane(v.z) & 511;
        return r;
    }

    // The item's output is stored: a gate/up tile is counted once every
    // wave's stores have reached memory.  Past the barrier every LDS read of the
    // item is done.  Wave 0 looks the requested ticket's item up before it, while
    // the other waves still store; where that ticket comes to nothing, the next
    // item is looked for after the count, since the down items wait for it.
    __device__ __forceinline__ void done(ArgSched &s, SchedLds &l, int phases, ArgTiles &ct)
    {
        have = pending < 0;
        if (have && fresh_tid() < 64) {
            Items q;
            q.load<LARGE, OWN>(l, phases, ct);
            const int it = take_requested(l, q);
            if (it >= 0) set_next(s, l, q, it);
            l.ahead = it >= 0;
        }
        if (!down) __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));   // vmcnt(0)
        __syncthreads();
        if (!down && fresh_tid() == 0) {
            int c = rti;
            if (OWN && l.hdr[4] != 0) c = l.rt[c].w;   // (at most kSchedLdsTiles row tiles then)
            agent_add(&s.dep[c * kDepStride], 1);
        }
    }
};

}  // namespace moe
