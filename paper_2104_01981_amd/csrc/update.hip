// The floating-point side of the ECRM update, on items already grouped by row (sort.hip):
//
//   apply_stripes   for each touched entry walk its updates in arrival order (Adagrad, Sec. 3.3.1),
//                   store the entry and its accumulator once, and add the entry's total difference in
//                   value and in accumulator to the stripe's parity rows (difference propagation,
//                   Sec. 3.3.2), which are read and written once per call.  The differences of one
//                   call telescope, so adding their sum is the same as adding them one by one.
//                   Entries that receive more than kLongRun updates in one call (the head of a skewed
//                   key distribution) are not walked here: their totals come from chains.hip.
//
//   route, count_rows: the smaller kernels of the path.
//
// One wavefront works on one row at a time: 64 lanes x float2 = a 128-float slice, so a load
// instruction of the wave moves 512 contiguous bytes from a wave-uniform (scalar) row address, and
// all control flow is wave-uniform.  All chain arithmetic is carried in fp64.  The kernels are
// templated on the update rule (struct Rule in rows.h): Adagrad or momentum SGD, updates of an entry
// applied one by one or combined; the description above is the Adagrad, one-by-one case.
#include "rows.h"

namespace ecrm {

// ================================================================================================
// apply
// ================================================================================================

constexpr uint32_t kGroupsPerTicket = 8, kNarrowGroupsPerTicket = 16;
constexpr int kListThreads = 256;
constexpr uint32_t kListMaxTiles = 4;
// A stripe of more updates than this goes to the end of the list, which the apply kernel takes first.  64 costs the list
// kernel time and gains the apply kernel nothing; 1024 leaves half of the gain (skewed batch of 2^24:
// 2363, 2266 and 2264 us with 1024, 256 and 64).
constexpr uint32_t kSlowStripe = 256;

// Lists the groups of kChunk sorted positions in which a stripe begins: the groups the apply kernel has work
// for.  All others lie inside runs -- every group of a long row's positions but its first -- and while
// they were handed out like the rest, the waves went through such a stretch at the pace of the ticket counter,
// a few nanoseconds per ticket with nothing done (1.2 of 8.4 ms on a Zipf batch).  A block looks at `tiles`
// tiles of kListThreads groups: a tile's positions are read coalesced, all loads of a thread in flight
// together, and their stripe numbers staged in LDS; a position whose stripe differs from its left neighbour's
// marks its group; the marked groups are appended to the list with one counter update per block (the list
// ascends inside a block's part; the order of the parts does not matter).  Groups with a long stripe are listed from
// the array's end (hdr->n_heavy of them).
__global__ __launch_bounds__(kListThreads) void active_groups_kernel(const uint32_t *sk, uint32_t n, Header *hdr,
                                                                     Divider dk, uint32_t tiles, uint32_t *active, uint32_t cap)
{
    constexpr uint32_t kTilePos = kListThreads * kChunk;                   // positions of a tile
    constexpr uint32_t kNone = 0xFFFFFFFFu, kEdge = 0xFFFFFFFEu;           // no stripe has these numbers
    __shared__ uint32_t s_q[1 + kTilePos];                                 // [0]: the position left of the tile
    __shared__ uint32_t s_mark[kListMaxTiles][kListThreads];
    __shared__ uint32_t s_cnt[kListMaxTiles][kListThreads / kWave];
    __shared__ uint32_t s_base, s_nslow, s_slow_base;
    if (hdr->batch_bad) return;
    n = min(n, hdr->n_valid);
    const uint32_t tid = threadIdx.x, lane = lane_id(), w = tid / kWave;
    uint32_t slow_mask = 0;                                                // bit t: group (t, tid) has a long stripe
    if (tid == 0) s_nslow = 0;
    const uint32_t g0 = blockIdx.x * tiles * (uint32_t)kListThreads;       // the block's first group
    for (uint32_t t = 0; t < tiles; ++t) {
        const uint32_t p_lo = (g0 + t * (uint32_t)kListThreads) * kChunk;  // < n + 2^16: no overflow, n <= 2^31
        uint32_t key[kChunk];
#pragma unroll
        for (uint32_t i = 0; i < kChunk; ++i) {
            const uint32_t p = p_lo + i * (uint32_t)kListThreads + tid;
            key[i] = p < n ? sk[p] : kNone;
        }
        // the stripe at the group's last position is the last that begins in it, if one does; the others end inside it
        const uint32_t rel_last = tid * kChunk + kChunk - 1u, far = rel_last + kSlowStripe;
        uint32_t far_key = kNone;
        if (far >= kTilePos && p_lo + far < n) far_key = sk[p_lo + far];
        if (tid == 0) s_q[0] = (p_lo > 0 && p_lo <= n) ? dk.div(sk[p_lo - 1]) : kEdge;
#pragma unroll
        for (uint32_t i = 0; i < kChunk; ++i)
            s_q[1 + i * (uint32_t)kListThreads + tid] = key[i] == kNone ? kNone : dk.div(key[i]);
        s_mark[t][tid] = 0;
        __syncthreads();
#pragma unroll
        for (uint32_t i = 0; i < kChunk; ++i) {
            const uint32_t rel = i * (uint32_t)kListThreads + tid;
            const uint32_t q = s_q[1 + rel];
            if (q != kNone && q != s_q[rel]) s_mark[t][rel / kChunk] = 1u;  // every writer writes 1
        }
        const uint32_t q_far = far < kTilePos ? s_q[1 + far] : far_key == kNone ? kNone : dk.div(far_key);
        if (q_far != kNone && q_far == s_q[1 + rel_last]) slow_mask |= 1u << t;
        __syncthreads();                                                   // s_q is free for the next tile
    }
    // compaction of the block's marks: per wave and tile a count, then one place in the list for the block
    uint32_t mine_mask = 0;                                                // bit t: group (t, tid) is marked
    for (uint32_t t = 0; t < tiles; ++t) {
        const bool marked = s_mark[t][tid] != 0, mine = marked && !((slow_mask >> t) & 1u);
        if (!marked) slow_mask &= ~(1u << t);
        const unsigned long long bal = __ballot(mine);
        if (mine) mine_mask |= 1u << t;
        if (lane == 0) s_cnt[t][w] = (uint32_t)__popcll(bal);
    }
    const uint32_t slow_at = slow_mask ? atomicAdd(&s_nslow, (uint32_t)__popc(slow_mask)) : 0u;
    __syncthreads();
    uint32_t total = 0, before[kListMaxTiles];
#pragma unroll
    for (uint32_t t = 0; t < kListMaxTiles; ++t) {
        before[t] = 0;
        if (t < tiles) {
#pragma unroll
            for (int v = 0; v < kListThreads / kWave; ++v) {
                const uint32_t c = s_cnt[t][v];
                if ((uint32_t)v == w) before[t] = total;
                total += c;
            }
        }
    }
    if (tid == 0) s_base = total ? atomicAdd(&hdr->n_active, total) : 0u;
    if (tid == kWave) s_slow_base = s_nslow ? atomicAdd(&hdr->n_heavy, s_nslow) : 0u;
    __syncthreads();
    for (uint32_t at = s_slow_base + slow_at; slow_mask; slow_mask &= slow_mask - 1u, ++at)
        active[cap - 1u - at] = g0 + (uint32_t)__builtin_ctz(slow_mask) * (uint32_t)kListThreads + tid;
#pragma unroll
    for (uint32_t t = 0; t < kListMaxTiles; ++t) {
        const bool mine = (mine_mask >> t) & 1u;                           // never set for t >= tiles
        const unsigned long long bal = __ballot(mine);
        if (mine) active[s_base + before[t] + (uint32_t)__popcll(bal & bits_below(lane))] = g0 + t * (uint32_t)kListThreads + tid;
    }
}

struct ApplyArgs {
    float *E, *A, *PE, *PA;
    const float *grads;
    const uint32_t *sk, *si;
    const uint32_t *active;      // groups of sorted positions in which a stripe begins, hdr->n_active from the front and
                                 // hdr->n_heavy, with a long stripe, from the end; null: no list was made, every group
                                 // is looked at
    uint32_t groups;             // room in the list
    const uint32_t *long_slot, *long_len;
    const double *long_res;
    Header *hdr;
    const unsigned long long *cnt;
    unsigned long long *load_data, *load_parity;
    uint32_t n;
    Geometry geo;
};

// General path, U gradients in flight: as many as cost no registers beside the window path's.  The stripe whose first item sits at sorted position `pos` (wave-uniform), walked
// through memory.  Used when the stripe does not fit the wave's window: runs of more than a few
// dozen updates, and entries whose totals come from the split-chain path.
template <int NC, int MODE, bool PARITY, int U = 8>
__device__ __forceinline__ void apply_stripe_general(const ApplyArgs &a, uint32_t n, uint32_t pos, uint32_t cb)
{
    const uint32_t D = a.geo.D, k = a.geo.k;
    const RuleParams rp = rule_params(a.geo);
    const uint32_t col0 = cb * NC * 128u;
    uint32_t key = uniform(a.sk[pos]);
    const uint32_t g = key / k;
    const rsrc_t perow = row_f32(a.PE, g, D, col0), parow = row_f32(a.PA, g, D, col0);

    D2 pe[NC], pa[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        pe[i] = PARITY ? widen2(ld2(perow, i)) : D2{0, 0};
        pa[i] = PARITY ? widen2(ld2(parow, i)) : D2{0, 0};
    }
    uint32_t cur = pos;
    do {
        const uint32_t x = key;                      // a new entry of this stripe starts at cur
        const bool is_long = (cur + kLongRun < n) && (uniform(a.sk[cur + kLongRun]) == x);
        const rsrc_t erow = row_f32(a.E, x, D, col0), arow = row_f32(a.A, x, D, col0);
        float2 e[NC], a0[NC];
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            e[i] = ld2(erow, i);
            a0[i] = ld2(arow, i);
        }
        D2 G[NC], acc[NC];
        if (is_long) {
            const uint32_t slot = uniform(a.long_slot[cur]);
            const rsrc_t r0 = row_f64(a.long_res, (size_t)slot * 2 + 0, D, col0);
            const rsrc_t r1 = row_f64(a.long_res, (size_t)slot * 2 + 1, D, col0);
#pragma unroll
            for (int i = 0; i < NC; ++i) {
                if (Rule<MODE>::combine) {           // slot 0 holds the sum of the run's gradients
                    G[i] = ldd2(r0, i);
                    acc[i] = D2{0, 0};
                } else {                             // slot 0: sum of the steps, slot 1: state after the run
                    acc[i] = ldd2(r0, i);
                    G[i] = ldd2(r1, i);
                }
            }
            cur += uniform(a.long_len[slot]);
        } else {
#pragma unroll
            for (int i = 0; i < NC; ++i) {
                G[i] = start2<MODE>(widen2(a0[i]));
                acc[i] = D2{0, 0};
            }
            // the run is at most kLongRun long: walk it 64 positions at a time, U gradients in flight
            bool done = false;
            while (!done) {
                const uint32_t lane = lane_id();
                const uint32_t wk = cur + lane < n ? a.sk[cur + lane] : kNoKey;
                const uint32_t wi = cur + lane < n ? a.si[cur + lane] : 0u;
                const unsigned long long other = ~__ballot(wk == x);
                const uint32_t cnt = other ? lowest_bit(other) : (uint32_t)kWave;   // leading run of x
                done = cnt < kWave;
                for (uint32_t u0 = 0; u0 < cnt; u0 += U) {
                    float2 gr[U][NC];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const uint32_t idx = from_lane(wi, min(u0 + u, cnt - 1));
                        const rsrc_t r = row_f32(a.grads, idx, D, col0);
#pragma unroll
                        for (int i = 0; i < NC; ++i) gr[u][i] = ldg2(r, i);
                    }
                    asm volatile("" ::: "memory");       // all of them now: each would be moved to where it is used
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (u0 + u < cnt) {
#pragma unroll
                            for (int i = 0; i < NC; ++i) item2<MODE>(G[i], acc[i], gr[u][i], rp);
                        }
                }
                cur += cnt;
            }
        }
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const D2 e64 = widen2(e[i]), a64 = widen2(a0[i]);
            finish2<MODE>(G[i], acc[i], a64, rp);
            st2(erow, i, narrow2(D2{e64.x - acc[i].x, e64.y - acc[i].y}));
            st2(arow, i, narrow2(G[i]));
            pe[i].x -= acc[i].x;
            pe[i].y -= acc[i].y;
            pa[i].x += G[i].x - a64.x;
            pa[i].y += G[i].y - a64.y;
        }
        key = cur < n ? uniform(a.sk[cur]) : kNoKey;
    } while (cur < n && key / k == g);

    if (PARITY) {
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            st2(perow, i, narrow2(pe[i]));
            st2(parow, i, narrow2(pa[i]));
        }
    }
}

#ifndef ECRM_PREFETCH
#define ECRM_PREFETCH 1
#endif
constexpr int kPrefetch = ECRM_PREFETCH;   // entries whose loads are issued ahead of the one being computed

// Loads of one entry's work: its row of E and A, its first gradient, and -- when it opens a
// stripe -- the stripe's parity rows.
template <int NC>
struct RowLoads {
    float2 e[NC], a[NC], g[NC], pe[NC], pa[NC];
    uint32_t x, j;
    bool opens;
};

template <int NC, bool PARITY>
__device__ __forceinline__ void issue_row(RowLoads<NC> &r, const ApplyArgs &a, uint32_t col0, uint32_t wkey,
                                          uint32_t widx, unsigned long long stripeheads, uint32_t j)
{
    const uint32_t D = a.geo.D;
    r.j = j;
    r.x = from_lane(wkey, j);
    r.opens = (stripeheads >> j) & 1ull;
    const uint32_t idx = from_lane(widx, j);
    const rsrc_t arow = row_f32(a.A, r.x, D, col0), grow = row_f32(a.grads, idx, D, col0),
                 erow = row_f32(a.E, r.x, D, col0);
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        r.a[i] = ld2(arow, i);
        r.g[i] = ldg2(grow, i);
        r.e[i] = ld2(erow, i);
        r.pe[i] = r.pa[i] = float2{0, 0};
    }
    if (PARITY && r.opens) {
        const uint32_t g = r.x / a.geo.k;
        const rsrc_t perow = row_f32(a.PE, g, D, col0), parow = row_f32(a.PA, g, D, col0);
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            r.pe[i] = ld2(perow, i);
            r.pa[i] = ld2(parow, i);
        }
    }
}

// Window path: every stripe that opens in the first kChunk lanes of the wave's 64-position window
// and ends inside the window.  Entries are taken one after the other; the loads of the next entry
// are issued before the current one is computed, so two entries' rows are in flight per wave.
template <int NC, int MODE, bool PARITY>
__device__ __forceinline__ void apply_window(const ApplyArgs &a, uint32_t wkey, uint32_t widx,
                                             unsigned long long rowheads, unsigned long long stripeheads,
                                             uint32_t first, uint32_t end, uint32_t cb)
{
    const uint32_t D = a.geo.D, k = a.geo.k;
    const RuleParams rp = rule_params(a.geo);
    const uint32_t col0 = cb * NC * 128u;
    unsigned long long todo = rowheads & bits_below(end) & ~bits_below(first);
    if (!todo) return;
    RowLoads<NC> q[kPrefetch];                        // entries whose loads are in flight, in order
    int qn = 0;
#pragma unroll
    for (int s = 0; s < kPrefetch; ++s) {
        if (todo) {
            issue_row<NC, PARITY>(q[s], a, col0, wkey, widx, stripeheads, lowest_bit(todo));
            todo &= todo - 1ull;
            qn = s + 1;
        }
    }
    D2 pe[NC], pa[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) pe[i] = pa[i] = D2{0, 0};
    while (true) {
        const RowLoads<NC> cur = q[0];
#pragma unroll
        for (int s = 0; s + 1 < kPrefetch; ++s) q[s] = q[s + 1];
        --qn;
        if (todo) {
            issue_row<NC, PARITY>(q[kPrefetch - 1], a, col0, wkey, widx, stripeheads, lowest_bit(todo));
            todo &= todo - 1ull;
            ++qn;                                     // the queue was full before the pop: slot kPrefetch-1 is free
        }
        const bool has_next = qn > 0;
        const uint32_t rend = has_next ? q[0].j : end;
        const bool next_opens = has_next && q[0].opens;
        D2 G[NC], acc[NC];
        float2 gr[NC];
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            G[i] = start2<MODE>(widen2(cur.a[i]));
            acc[i] = D2{0, 0};
            gr[i] = cur.g[i];
        }
#ifndef ECRM_ITEM_AHEAD
#define ECRM_ITEM_AHEAD 4
#endif
        // The entry's updates, in arrival order.  The gradients of the next few updates are in flight
        // while one is applied: with one in flight a run of m updates cost m memory latencies, which
        // is what bounded the workloads with several updates per entry (4 in flight: -3 % and -5 % on
        // large_uniform and medium; two for D > 128, where more would cost a wave per SIMD).
        constexpr int AH = (NC == 1 ? ECRM_ITEM_AHEAD : 2) - 1;
        float2 nx[AH][NC];
#pragma unroll
        for (int q = 0; q < AH; ++q) {
#pragma unroll
            for (int i = 0; i < NC; ++i) nx[q][i] = float2{0, 0};
            if (cur.j + 1 + q < rend) {
                const rsrc_t r = row_f32(a.grads, from_lane(widx, cur.j + 1 + q), D, col0);
#pragma unroll
                for (int i = 0; i < NC; ++i) nx[q][i] = ldg2(r, i);
            }
        }
        for (uint32_t t = cur.j;;) {
            float2 in[NC];
#pragma unroll
            for (int i = 0; i < NC; ++i) in[i] = float2{0, 0};
            if (t + 1 + AH < rend) {
                const rsrc_t r = row_f32(a.grads, from_lane(widx, t + 1 + AH), D, col0);
#pragma unroll
                for (int i = 0; i < NC; ++i) in[i] = ldg2(r, i);
            }
#pragma unroll
            for (int i = 0; i < NC; ++i) item2<MODE>(G[i], acc[i], gr[i], rp);
            if (t + 1 >= rend) break;
#pragma unroll
            for (int i = 0; i < NC; ++i) {
                gr[i] = nx[0][i];
#pragma unroll
                for (int q = 0; q + 1 < AH; ++q) nx[q][i] = nx[q + 1][i];
                nx[AH - 1][i] = in[i];
            }
            ++t;
        }
        if (cur.opens) {
#pragma unroll
            for (int i = 0; i < NC; ++i) {
                pe[i] = widen2(cur.pe[i]);
                pa[i] = widen2(cur.pa[i]);
            }
        }
        const rsrc_t erow = row_f32(a.E, cur.x, D, col0), arow = row_f32(a.A, cur.x, D, col0);
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const D2 e64 = widen2(cur.e[i]), a64 = widen2(cur.a[i]);
            finish2<MODE>(G[i], acc[i], a64, rp);
            st2(erow, i, narrow2(D2{e64.x - acc[i].x, e64.y - acc[i].y}));
            st2(arow, i, narrow2(G[i]));
            pe[i].x -= acc[i].x;
            pe[i].y -= acc[i].y;
            pa[i].x += G[i].x - a64.x;
            pa[i].y += G[i].y - a64.y;
        }
        if (PARITY && (!has_next || next_opens)) {    // last entry of its stripe: the parity rows are complete
            const uint32_t g = cur.x / k;
            const rsrc_t perow = row_f32(a.PE, g, D, col0), parow = row_f32(a.PA, g, D, col0);
#pragma unroll
            for (int i = 0; i < NC; ++i) {
                st2(perow, i, narrow2(pe[i]));
                st2(parow, i, narrow2(pa[i]));
            }
        }
        if (!has_next) break;
    }
}

// The same for rows of at most 64 (P = 2) or 32 (P = 4) floats: a step takes up to P consecutive entries, one to each group of
// 64 / P lanes, so that one instruction moves P rows; with one row to a wave half of the lanes, or more, had nothing to do, and
// the instructions, not the memory, set the pace.  Half-Zipf momentum updates, k = 2, this kernel alone in a trace, and the whole
// call: 1.5 M of 64 floats 537 us, now 354 to 434 with the placement of the tables, the call 721, now 587; of 32 floats 492, now
// 258, the call 680, now 410; 3 M of 16 floats 621, now 355, the call 853, now 547.  All control flow is that of the wave: the
// entries' numbers of updates and stripes differ from group to group, and what a group has no part in is masked; every exchange
// between groups is executed by all lanes.  Rows are read through per-lane addresses.
template <int P>
struct NarrowLoads {
    float2 e, a, g, pe, pa;
    uint32_t x, j, cnt;          // the group's entry: row, first position of the window, updates (0: no entry)
    bool opens, closes;          // the first, the last entry of its stripe
    uint32_t most, groups;       // of the step (wave-uniform): updates of its longest entry, entries
};

__device__ __forceinline__ float2 load2(const float *p)
{
    typedef float f2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(float2, __builtin_nontemporal_load((const f2 *)p));
}
__device__ __forceinline__ void store2(float *p, float2 v)
{
    typedef float f2 __attribute__((ext_vector_type(2)));
    __builtin_nontemporal_store(__builtin_bit_cast(f2, v), (f2 *)p);
}

// takes the next entries from todo (not empty)
template <int P, bool PARITY>
__device__ __forceinline__ void issue_narrow(NarrowLoads<P> &r, const ApplyArgs &a, uint32_t col, uint32_t wkey, uint32_t widx,
                                             unsigned long long stripeheads, unsigned long long &todo, uint32_t end)
{
    const uint32_t D = a.geo.D, mine = lane_id() / (kWave / P);
    r.most = r.groups = 0;
    r.cnt = 0;
    r.x = r.j = 0;
    r.opens = r.closes = false;
#pragma unroll
    for (uint32_t q = 0; q < (uint32_t)P; ++q) {
        if (!todo) break;
        const uint32_t j = lowest_bit(todo);
        todo &= todo - 1ull;
        const uint32_t next = todo ? lowest_bit(todo) : end, x = from_lane(wkey, j);
        const bool opens = (stripeheads >> j) & 1ull, closes = !todo || ((stripeheads >> next) & 1ull);
        r.most = max(r.most, next - j);
        r.groups = q + 1u;
        // the groups behind the last entry load its rows as well, and leave them alone
        r.x = mine >= q ? x : r.x;
        r.j = mine >= q ? j : r.j;
        r.cnt = mine == q ? next - j : mine > q ? 0u : r.cnt;
        r.opens = mine == q ? opens : mine > q ? false : r.opens;
        r.closes = mine == q ? closes : mine > q ? false : r.closes;
    }
    const uint32_t idx = __shfl(widx, (int)r.j, kWave);
    r.a = load2(a.A + (size_t)r.x * D + col);
    r.g = load2(a.grads + (size_t)idx * D + col);
    r.e = load2(a.E + (size_t)r.x * D + col);
    r.pe = r.pa = float2{0, 0};
    if (PARITY && r.opens) {
        const size_t at = (size_t)a.geo.dk.div(r.x) * D + col;
        r.pe = load2(a.PE + at);
        r.pa = load2(a.PA + at);
    }
}

template <int P, int MODE, bool PARITY>
__device__ __forceinline__ void apply_window_narrow(const ApplyArgs &a, uint32_t wkey, uint32_t widx, unsigned long long rowheads,
                                                    unsigned long long stripeheads, uint32_t first, uint32_t end)
{
    constexpr uint32_t kLanes = kWave / P;
    const uint32_t D = a.geo.D, lane = lane_id(), group = lane / kLanes, col_lane = lane % kLanes;
    const bool live = 2u * col_lane < D;                   // D is a multiple of 4: both columns or none
    const uint32_t col = live ? 2u * col_lane : 0u;
    const RuleParams rp = rule_params(a.geo);
    unsigned long long todo = rowheads & bits_below(end) & ~bits_below(first);
    if (!todo) return;
    NarrowLoads<P> next;
    issue_narrow<P, PARITY>(next, a, col, wkey, widx, stripeheads, todo, end);
    D2 pe = D2{0, 0}, pa = D2{0, 0};                       // parity rows of the stripe that goes on into the next step
    for (bool more = true; more;) {
        const NarrowLoads<P> cur = next;
        more = todo != 0;
        if (more) issue_narrow<P, PARITY>(next, a, col, wkey, widx, stripeheads, todo, end);
        D2 G = start2<MODE>(widen2(cur.a)), acc = D2{0, 0};
        // the entries' updates, those of the next few in flight (apply_window); past an entry's end: its last one again
        constexpr int AH = ECRM_ITEM_AHEAD - 1;
        const uint32_t last = cur.j + max(cur.cnt, 1u) - 1u;
        float2 gr = cur.g, nx[AH];
        auto gradient = [&](uint32_t u) {
            const uint32_t idx = __shfl(widx, (int)min(cur.j + u, last), kWave);
            return load2(a.grads + (size_t)idx * D + col);
        };
#pragma unroll
        for (int q = 0; q < AH; ++q) {
            nx[q] = float2{0, 0};
            if (1u + q < cur.most) nx[q] = gradient(1u + q);
        }
        for (uint32_t u = 0;;) {
            float2 in = float2{0, 0};
            if (u + 1 + AH < cur.most) in = gradient(u + 1 + AH);
            if (u < cur.cnt) item2<MODE>(G, acc, gr, rp);
            if (++u >= cur.most) break;
            gr = nx[0];
#pragma unroll
            for (int q = 0; q + 1 < AH; ++q) nx[q] = nx[q + 1];
            nx[AH - 1] = in;
        }
        const D2 e64 = widen2(cur.e), a64 = widen2(cur.a);
        finish2<MODE>(G, acc, a64, rp);
        const bool mine = cur.cnt != 0 && live;
        if (mine) {
            store2(a.E + (size_t)cur.x * D + col, narrow2(D2{e64.x - acc.x, e64.y - acc.y}));
            store2(a.A + (size_t)cur.x * D + col, narrow2(G));
        }
        if (PARITY) {
            // from group to group: the parity rows as they are after the group's entry
            if (cur.opens) {
                pe = widen2(cur.pe);
                pa = widen2(cur.pa);
            }
            const D2 dpa = D2{G.x - a64.x, G.y - a64.y};
            D2 ve = D2{pe.x - acc.x, pe.y - acc.y}, va = D2{pa.x + dpa.x, pa.y + dpa.y};
#pragma unroll
            for (uint32_t q = 1; q < (uint32_t)P; ++q) {
                const int from = (int)((q - 1u) * kLanes + col_lane);
                const D2 fe = D2{__shfl(ve.x, from, kWave), __shfl(ve.y, from, kWave)};
                const D2 fa = D2{__shfl(va.x, from, kWave), __shfl(va.y, from, kWave)};
                if (group == q && !cur.opens) {
                    ve = D2{fe.x - acc.x, fe.y - acc.y};
                    va = D2{fa.x + dpa.x, fa.y + dpa.y};
                }
            }
            if (mine && cur.closes) {
                const size_t at = (size_t)a.geo.dk.div(cur.x) * D + col;
                store2(a.PE + at, narrow2(ve));
                store2(a.PA + at, narrow2(va));
            }
            const int from = (int)((cur.groups - 1u) * kLanes + col_lane);
            pe = D2{__shfl(ve.x, from, kWave), __shfl(ve.y, from, kWave)};
            pa = D2{__shfl(va.x, from, kWave), __shfl(va.y, from, kWave)};
        }
    }
}

// The groups of kChunk sorted positions in which a stripe begins (active_groups_kernel lists them) are handed out through a
// counter instead of by a fixed stride: the work per group varies (runs, long stripes), and with a fixed stride the
// slowest wave set the kernel's time (6.50 -> 6.22 ms).  One ticket covers kGroupsPerTicket listed groups: one group per
// ticket made the counter itself the bottleneck (12.5 ms), 64 per ticket is too coarse again.  A wave's first ticket is
// its own number (no counter traffic at start-up, which is all a small batch consists of); later ones come from the
// counter.  Small batches get smaller tickets, so that every wave has work: four to a wave, but no more than two once that
// would make a ticket shorter than half of the largest: a counter update takes as long as the memory takes to move a group or
// two (at least one group to a ticket, us a call: 600 000 uniform updates 585, now 465; 2 M Zipf, k = 10, 905, now 650; two
// tickets to a wave in larger batches as well: 2 M half Zipf 1160, then 1182).  Narrow rows, twice the groups: 3 M half-Zipf
// updates of 16 floats 570, now 547; 1.5 M Zipf of 48, combined, 449, now 372.  Groups with a long stripe come first, one to
// a ticket: one wave walks such a stripe for up to 150 us, and where it came late the others were idle meanwhile (apply
// kernels of Zipf and half-Zipf batches: 617 -> 535, 2226 -> 2110, 2390 -> 2263, 7770 -> 7672 us).
struct GroupTickets {
    uint32_t nslow, nact, per, ticket;
    bool first;
    __device__ __forceinline__ void init(const ApplyArgs &a, uint32_t n, uint32_t most)
    {
        const uint32_t ngroups = (n + kChunk - 1) / kChunk;
        nslow = a.active ? min(a.hdr->n_heavy, ngroups) : 0u;
        nact = a.active ? min(a.hdr->n_active, ngroups) : ngroups;   // no list (a small batch): every group
        const uint32_t waves = wave_count();
        per = max(max(min(most / 2u, (nact + 2u * waves - 1u) / (2u * waves)), min(most, nact / (4u * waves))), 1u);
        ticket = wave_id();
        first = true;
    }
    // the next ticket's groups: lane i < left holds the i-th
    __device__ __forceinline__ bool next(const ApplyArgs &a, uint32_t &listed, uint32_t &left)
    {
        const uint32_t lane = lane_id(), all = nslow + (nact + per - 1u) / per;
        if (!first) {
            if (all <= wave_count()) return false;
            uint32_t t = 0;
            if (lane == 0) t = atomicAdd(&a.hdr->apply_ticket, 1u);
            ticket = wave_count() + uniform(t);
        }
        first = false;
        if (ticket >= all) return false;
        if (ticket < nslow) {
            left = 1u;
            listed = a.active[a.groups - 1u - ticket];
        } else {
            const uint32_t at = (ticket - nslow) * per;
            left = min(per, nact - at);
            listed = lane < left ? (a.active ? a.active[at + lane] : at + lane) : 0u;
        }
        return true;
    }
};

// the batch is valid: publish its per-server counts
__device__ __forceinline__ void publish_counts(const ApplyArgs &a)
{
    if (blockIdx.x != 0) return;
    const uint32_t S = a.geo.S;
    for (uint32_t i = threadIdx.x; i < S; i += blockDim.x) {
        if (a.load_data) a.load_data[i] += a.cnt[i];
        if (a.load_parity) a.load_parity[i] += a.cnt[S + i];
    }
}

// What a wave finds in the 64 positions from a group's first: heads of rows and of stripes, and the range of the stripes
// that begin in the group and end in the window.
struct Window {
    unsigned long long rowheads, stripeheads;
    uint32_t first, end, last;
    bool any, last_inside;       // any: a stripe begins in the group; else nothing below holds.  The last one may go on.
};
__device__ __forceinline__ Window look_at(uint32_t wkey, uint32_t prevk, uint32_t p0, uint32_t n, uint32_t k)
{
    const uint32_t lane = lane_id();
    Window w;
    uint32_t leftk = __shfl_up(wkey, 1, kWave);
    if (lane == 0) leftk = prevk;
    const bool valid = wkey != kNoKey;
    const bool rh = !valid || leftk == kNoKey || leftk != wkey;    // lanes past n end the last run
    const bool sh = valid && (leftk == kNoKey || leftk / k != wkey / k);
    w.rowheads = __ballot(rh);
    w.stripeheads = __ballot(sh);
    const uint32_t vend = min((uint32_t)kWave, n - p0);
    const unsigned long long owned = w.stripeheads & bits_below(kChunk);
    w.any = owned != 0;
    w.first = w.any ? lowest_bit(owned) : 0u;
    w.last = w.any ? 63u - (uint32_t)__builtin_clzll(owned) : 0u;
    const unsigned long long after = w.stripeheads & ~bits_below(w.last + 1);
    w.last_inside = after != 0ull || p0 + kWave >= n;
    w.end = w.last_inside ? (after ? lowest_bit(after) : vend) : w.last;
    return w;
}

// P: entries to a wave at a time
template <int NC, int MODE, bool PARITY, int P = 1>
__device__ __forceinline__ void apply_stripes_body(const ApplyArgs &a)
{
    if (a.hdr->batch_bad) return;
    publish_counts(a);
    const uint32_t n = min(a.n, a.hdr->n_valid), k = a.geo.k, lane = lane_id();
    GroupTickets tickets;
    tickets.init(a, n, P > 1 ? kNarrowGroupsPerTicket : kGroupsPerTicket);
    uint32_t left = 0, taken = 0, listed = 0;          // groups left in the ticket, taken from it; lane i: its group i
    uint32_t pf_ch = 0xFFFFFFFFu, pf_key = 0, pf_idx = 0, pf_prev = 0;
    for (;;) {
        if (left == 0) {
            if (!tickets.next(a, listed, left)) break;
            taken = 0;
        }
        const uint32_t ch = from_lane(listed, taken);
        ++taken;
        --left;
        const uint32_t p0 = ch * kChunk;
        uint32_t wkey, widx, prevk;
        // The group's 64 (row, index) pairs were asked for while the previous group was being worked on;
        // only a ticket's first group has to wait for them.
        if (pf_ch == ch) {
            wkey = pf_key;
            widx = pf_idx;
            prevk = uniform(pf_prev);
        } else {
            wkey = p0 + lane < n ? a.sk[p0 + lane] : kNoKey;
            widx = p0 + lane < n ? a.si[p0 + lane] : 0u;
            prevk = p0 ? uniform(a.sk[p0 - 1]) : kNoKey;
        }
        if (left > 0) {
            pf_ch = from_lane(listed, taken);
            const uint32_t q0 = pf_ch * kChunk;
            pf_key = q0 + lane < n ? a.sk[q0 + lane] : kNoKey;
            pf_idx = q0 + lane < n ? a.si[q0 + lane] : 0u;
            pf_prev = q0 ? a.sk[q0 - 1] : kNoKey;
        }
        const Window w = look_at(wkey, prevk, p0, n, k);
        if (!w.any) continue;
        if (P > 1) {
            apply_window_narrow<P, MODE, PARITY>(a, wkey, widx, w.rowheads, w.stripeheads, w.first, w.end);
            if (!w.last_inside) apply_stripe_general<NC, MODE, PARITY, 16>(a, n, p0 + w.last, 0);
            continue;
        }
        for (uint32_t cb = 0; cb < a.geo.ncb; ++cb) {
            apply_window<NC, MODE, PARITY>(a, wkey, widx, w.rowheads, w.stripeheads, w.first, w.end, cb);
            if (!w.last_inside) apply_stripe_general<NC, MODE, PARITY, NC == 1 ? 8 : 12>(a, n, p0 + w.last, cb);
        }
    }
}

// D <= 128: one 128-float slice per lane pair; D > 128: two slices per lane.  The narrow ones: D <= 64 (P = 2), D <= 32 (4).
template <int MODE>
__global__ __launch_bounds__(256) void apply_stripes_kernel_d128(ApplyArgs a)
{
    apply_stripes_body<1, MODE, true>(a);
}
template <int MODE>
__global__ __launch_bounds__(256) void apply_stripes_kernel_d256(ApplyArgs a)
{
    apply_stripes_body<2, MODE, true>(a);
}
template <int MODE, bool PARITY, int P>
__global__ __launch_bounds__(256) void apply_narrow_kernel(ApplyArgs a)
{
    apply_stripes_body<1, MODE, PARITY, P>(a);
}
// The same walk with the parity rows left alone: entries and their state only.  This is the update
// of a system without redundancy (the baseline the overheads of Sec. 4.3 are quoted against), and
// each of the two halves of the gradient-propagation strawman of Sec. 3.3.1.
template <int MODE>
__global__ __launch_bounds__(256) void apply_rows_kernel_d128(ApplyArgs a)
{
    apply_stripes_body<1, MODE, false>(a);
}
template <int MODE>
__global__ __launch_bounds__(256) void apply_rows_kernel_d256(ApplyArgs a)
{
    apply_stripes_body<2, MODE, false>(a);
}

// Combined (synchronous) rule: one update per modified entry, so the per-server load counts one per
// distinct row of the batch and one parity update for each (Sec. 3.6, Sec. 4.4).
__global__ __launch_bounds__(256) void count_rows_kernel(const uint32_t *sk, uint32_t n, Header *hdr,
                                                         unsigned long long *cnt, uint32_t k, uint32_t S)
{
    __shared__ uint32_t s_cnt[2 * 1024];
    if (hdr->batch_bad) return;
    n = min(n, hdr->n_valid);
    for (uint32_t i = threadIdx.x; i < 2 * S; i += blockDim.x) s_cnt[i] = 0;
    __syncthreads();
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t p = blockIdx.x * blockDim.x + threadIdx.x; p < n; p += stride) {
        const uint32_t x = sk[p];
        if (p == 0 || sk[p - 1] != x) {
            const uint32_t g = x / k, j = x - g * k;
            atomicAdd(&s_cnt[(g + 1 + j) % S], 1u);
            atomicAdd(&s_cnt[S + g % S], 1u);
        }
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < 2 * S; i += blockDim.x)
        if (s_cnt[i]) atomicAdd(&cnt[i], (unsigned long long)s_cnt[i]);
}

// ================================================================================================
// route
// ================================================================================================

__global__ __launch_bounds__(256) void route_kernel(const uint64_t *keys, uint64_t n, uint64_t rows, uint32_t k,
                                                    uint32_t S, uint64_t *stripe, uint32_t *member,
                                                    uint32_t *data_srv, uint32_t *parity_srv, Header *hdr)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const uint64_t x = keys[i];
        if (x >= rows) {
            atomicOr(&hdr->err_sticky, 1u);
            continue;
        }
        const uint64_t g = x / k;
        const uint32_t j = (uint32_t)(x - g * k);
        if (stripe) stripe[i] = g;
        if (member) member[i] = j;
        if (data_srv) data_srv[i] = (uint32_t)((g + 1 + j) % S);
        if (parity_srv) parity_srv[i] = (uint32_t)(g % S);
    }
}

// ================================================================================================
// host side
// ================================================================================================

// the apply kernel for rows of D floats
typedef void (*ApplyKernel)(ApplyArgs);
template <int NC, int MODE>
static ApplyKernel apply_kernel(uint32_t D, bool parity)
{
    if (D <= 32) return parity ? apply_narrow_kernel<MODE, true, 4> : apply_narrow_kernel<MODE, false, 4>;
    if (D <= 64) return parity ? apply_narrow_kernel<MODE, true, 2> : apply_narrow_kernel<MODE, false, 2>;
    if (NC == 1) return parity ? apply_stripes_kernel_d128<MODE> : apply_rows_kernel_d128<MODE>;
    return parity ? apply_stripes_kernel_d256<MODE> : apply_rows_kernel_d256<MODE>;
}

template <int NC, int MODE>
static bool apply_grids_for(uint32_t D, int cus, LaunchGrids *out)
{
    out->apply = resident_grid(apply_kernel<NC, MODE>(D, true), cus);
    out->rows = resident_grid(apply_kernel<NC, MODE>(D, false), cus);
    return out->apply > 0 && out->rows > 0;
}

template <int NC, int MODE>
static void apply_for(const ApplyArgs &a, const LaunchGrids &lg, bool parity, hipStream_t st)
{
    hipLaunchKernelGGL((apply_kernel<NC, MODE>(a.geo.D, parity)), dim3(parity ? lg.apply : lg.rows), dim3(256), 0, st, a);
}

bool query_launch_grids(const Geometry &g, int cus, LaunchGrids *out)
{
    bool ok = false;
    ECRM_DISPATCH(ok = apply_grids_for, g.D, cus, out);
    return ok && query_chain_grids(g, cus, out);
}

// A batch this small is one wave's ticket or two per wave anyway: the list would cost a launch and save nothing.
static bool lists_groups(uint32_t n) { return n > (1u << 18); }

// the list of groups launch_apply works from; n > 0
void launch_active_groups(const Scratch &s, const Geometry &g, const uint32_t *sk, uint32_t n, hipStream_t st)
{
    if (!lists_groups(n)) return;
    const uint32_t groups = (n + kChunk - 1) / kChunk;
    // a large batch: several tiles per block, so that the list's counter is not updated at its own pace
    const uint32_t tiles = groups > 64u * kListThreads ? kListMaxTiles : 1u;
    const uint32_t per_block = tiles * kListThreads;
    const dim3 grid((groups + per_block - 1) / per_block), block(kListThreads);
    hipLaunchKernelGGL(active_groups_kernel, grid, block, 0, st, sk, n, s.hdr, make_divider(g.k), tiles, s.active, groups);
}

void launch_apply(const Scratch &s, const Geometry &g, const LaunchGrids &lg, float *E, float *A, float *PE, float *PA,
                  unsigned long long *load_data, unsigned long long *load_parity, const float *grads,
                  const uint32_t *sk, const uint32_t *si, uint32_t n, int cus, hipStream_t st)
{
    const bool parity = PE != nullptr;      // no parity tables: entries and state only
    ApplyArgs a;
    a.E = E; a.A = A; a.PE = PE; a.PA = PA;
    a.grads = grads; a.sk = sk; a.si = si;
    a.long_slot = s.long_slot; a.long_len = s.long_len; a.long_res = s.long_res;
    a.active = lists_groups(n) ? s.active : nullptr;
    a.groups = (n + kChunk - 1) / kChunk;
    a.hdr = s.hdr; a.cnt = s.cnt;
    a.load_data = load_data; a.load_parity = load_parity;
    a.n = n; a.geo = g;
    if ((g.mode == kAdagradCombine || g.mode == kMomentumCombine) && load_data)      // one load count per modified entry
        hipLaunchKernelGGL(count_rows_kernel, dim3(cus * 8), dim3(256), 0, st, sk, n, s.hdr, s.cnt, g.k, g.S);
    ECRM_DISPATCH(apply_for, a, lg, parity, st);
}
#undef ECRM_DISPATCH

void launch_route(const Scratch &s, const Geometry &g, const uint64_t *keys, uint64_t n, uint64_t *stripe,
                  uint32_t *member, uint32_t *data_srv, uint32_t *parity_srv, hipStream_t st)
{
    uint64_t blocks = (n + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(route_kernel, dim3((uint32_t)blocks), dim3(256), 0, st, keys, n, (uint64_t)g.rows, g.k, g.S,
                       stripe, member, data_srv, parity_srv, s.hdr);
}

}  // namespace ecrm
