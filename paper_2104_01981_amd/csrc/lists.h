// Stripes from a sorted list of (row, position) pairs in LDS, by a workgroup of kBucketThreads: the walk over a window of the
// list, the walk of a stripe that is longer than that, sorting, and handing the list out to the waves.  Shared by the kernels of
// small batches (buckets.hip, direct.hip).
#pragma once

#include "long_runs.h"

namespace ecrm {

typedef unsigned long long u64;

constexpr int kBucketWaves = kBucketThreads / kWave;
// Updates of a run from which on the waves of a workgroup share its columns; and it has to be a third of its stripe: of more
// runs of a kind the waves take one each (2^19 updates on 2^14 rows, 128 to a stripe: 161 us with every run's columns
// shared, 124 so; on 2^13 rows of 512 floats 402 and 292).
constexpr uint32_t kTogether = 32;
__device__ __forceinline__ uint32_t together(uint32_t stripe) { return max(kTogether, stripe / 3u); }

__device__ __forceinline__ uint32_t item_row(u64 it) { return (uint32_t)(it >> 32); }

// exclusive scan of one value per thread over a workgroup of WAVES waves
template <int WAVES = kBucketWaves>
__device__ __forceinline__ uint32_t bucket_excl_scan(uint32_t v, uint32_t *s_wave, uint32_t &total)
{
    const uint32_t lane = lane_id(), wave = threadIdx.x / kWave;
    uint32_t incl = v;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t t = __shfl_up(incl, d, kWave);
        if (lane >= (uint32_t)d) incl += t;
    }
    if (lane == kWave - 1) s_wave[wave] = incl;
    __syncthreads();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        const uint32_t t = s_wave[w];
        if ((uint32_t)w < wave) off += t;
        tot += t;
    }
    __syncthreads();
    total = tot;
    return off + incl - v;
}

struct RowArgs {
    float *E, *A, *PE, *PA;
    const float *grads;
    Geometry geo;
};

// ================================================================================================
// the walk over a window of sorted (row, gradient row) pairs
// ================================================================================================

// One step of the walk takes up to U consecutive updates of one entry.  What it needs from memory: their gradients; the
// rows of E and A if the first of them is its entry's first; the parity rows if the entry opens a stripe.  Rows that are
// not needed are asked for through a buffer resource of size zero, which returns zeros without touching memory: every
// step issues the same loads, so the compiler knows how many are younger than the ones it waits for, and the loads of
// Q steps really are in flight.  (With the loads under branches, as in the apply kernel of large batches, it waits for
// everything before each entry; there the 24 waves of a compute unit hide that, here there are too few of them.  A load
// of size zero still takes its 17 cycles of the compute unit's memory pipe, which a batch of this size can afford and
// the large ones cannot: 2^22 updates in 963 us with branches, 1300 us with steps of one update.)
template <int NC, int U>
struct StepLoads {
    float2 a[NC], e[NC], g[U][NC], pe[NC], pa[NC];
};

// The chain of the entry in work and the parity rows of its stripe.  A step that brings no rows leaves those of the entry
// and the stripe in work as they are: taking a set of loads in is a select and needs no branch (added to zeros instead, a
// stored -0.0 became +0.0).
template <int NC>
struct Walk {
    D2 G[NC], acc[NC], pe[NC], pa[NC];
    float2 e[NC], a[NC];
    __device__ __forceinline__ void begin()
    {
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            pe[i] = pa[i] = D2{-0.0, -0.0};            // the neutral summand
            e[i] = a[i] = float2{0, 0};
        }
        clear_chain();
    }
    __device__ __forceinline__ void clear_chain()
    {
#pragma unroll
        for (int i = 0; i < NC; ++i) G[i] = acc[i] = D2{0, 0};
    }
};

__device__ __forceinline__ rsrc_t row_if(const float *table, uint32_t row, uint32_t D, uint32_t col0, bool wanted)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(table + (size_t)row * D + col0), 0,
                                             wanted ? (int)((D - col0) * 4u) : 0, kRsrcFlags);
}

// Issues the loads of the step that starts in lane t; returns how many updates it takes (0: nothing is left).
template <int NC, int U, bool PARITY>
__device__ __forceinline__ uint32_t issue_step(StepLoads<NC, U> &l, const RowArgs &a, uint32_t col0, uint32_t wkey,
                                               uint32_t widx, u64 rowheads, u64 stripeheads, uint32_t t, uint32_t end)
{
    const uint32_t D = a.geo.D, lane = min(t, (uint32_t)kWave - 1u);
    const bool in = t < end, head = in && ((rowheads >> lane) & 1ull), opens = in && ((stripeheads >> lane) & 1ull);
    const u64 next = rowheads & ~bits_below(lane + 1u);
    const uint32_t run_end = next ? min(lowest_bit(next), end) : end;
    const uint32_t cnt = in ? min((uint32_t)U, run_end - t) : 0u;
    const uint32_t x = from_lane(wkey, lane);
    const rsrc_t arow = row_if(a.A, x, D, col0, head), erow = row_if(a.E, x, D, col0, head);
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        l.a[i] = ld2(arow, i);
        l.e[i] = ld2(erow, i);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const rsrc_t grow = row_if(a.grads, from_lane(widx, min(t + u, (uint32_t)kWave - 1u)), D, col0, (uint32_t)u < cnt);
#pragma unroll
        for (int i = 0; i < NC; ++i) l.g[u][i] = ldg2(grow, i);
    }
    if (PARITY) {
        const uint32_t g = a.geo.dk.div(x);
        const rsrc_t perow = row_if(a.PE, g, D, col0, opens), parow = row_if(a.PA, g, D, col0, opens);
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            l.pe[i] = ld2(perow, i);
            l.pa[i] = ld2(parow, i);
        }
    }
    return cnt;
}

// What a wave's part of a list that is cut at entries has of stripes that are not all its own.
struct Shared {
    bool before, goes_on;      // the first entries belong to a stripe that another wave opens; another wave goes on with the last one
    double *part;              // for the differences of those first entries
};

// The updates in lanes [first, end) of a window, in order: whole stripes; or (SPLIT) whole entries, where the differences of a
// stripe that another wave opens are left in from.part, and one that another wave goes on with is not stored: if this wave has
// opened it, w has its parity rows so far.
template <int NC, int MODE, bool PARITY, int Q, int U, bool SPLIT>
__device__ __forceinline__ void walk_window(const RowArgs &a, uint32_t wkey, uint32_t widx, u64 rowheads, u64 stripeheads,
                                            uint32_t first, uint32_t end, uint32_t cb, Walk<NC> &w, Shared from)
{
    const uint32_t D = a.geo.D;
    const RuleParams rp = rule_params(a.geo);
    const uint32_t col0 = cb * NC * 128u;
    w.begin();
    StepLoads<NC, U> l[Q];
    uint32_t at[Q], cnt[Q], next = first;          // lane a step in flight starts in, and how many updates it takes
#pragma unroll
    for (int s = 0; s < Q; ++s) {
        at[s] = next;
        cnt[s] = issue_step<NC, U, PARITY>(l[s], a, col0, wkey, widx, rowheads, stripeheads, next, end);
        next += cnt[s];
        asm volatile("" ::: "memory");             // in this order: the first set is waited for first
        __builtin_amdgcn_sched_barrier(0);
    }
    // No way out of the loop but its end: an exit in the middle would let the compiler see a path into the next round
    // with fewer loads behind the first set's.  Steps past the end take zeros in and compute nothing.
    while (cnt[0]) {
#pragma unroll
        for (int s = 0; s < Q; ++s) {
            const bool head = cnt[s] && ((rowheads >> at[s]) & 1ull), opens = cnt[s] && ((stripeheads >> at[s]) & 1ull);
#pragma unroll
            for (int i = 0; i < NC; ++i) {
                w.a[i].x = head ? l[s].a[i].x : w.a[i].x;
                w.a[i].y = head ? l[s].a[i].y : w.a[i].y;
                w.e[i].x = head ? l[s].e[i].x : w.e[i].x;
                w.e[i].y = head ? l[s].e[i].y : w.e[i].y;
                // In registers of their own: where they stayed in those of the loads, the next loads of two slices went to
                // others and were copied, and waited for, at the end of the loop (one slice has no such copies).  Of 33
                // batches of 4096 to 300 000 updates, rows of 132 to 1024 floats, all three rules, none lost and most gained, up to 4 %:
                // 65 536 uniform on 2^14 rows of 132, 256, 512 floats 64.7 -> 62.3, 67.7 -> 65.3, 114.6 -> 110.2 us.
                if (NC > 1) {
                    const float2 a0 = w.a[i], e0 = w.e[i];
                    asm volatile("v_mov_b32 %0, %4\n\tv_mov_b32 %1, %5\n\tv_mov_b32 %2, %6\n\tv_mov_b32 %3, %7"
                                 : "=&v"(w.a[i].x), "=&v"(w.a[i].y), "=&v"(w.e[i].x), "=&v"(w.e[i].y)
                                 : "v"(a0.x), "v"(a0.y), "v"(e0.x), "v"(e0.y));
                }
                if (!Rule<MODE>::combine) {
                    w.G[i].x = head ? (double)l[s].a[i].x : w.G[i].x;
                    w.G[i].y = head ? (double)l[s].a[i].y : w.G[i].y;
                }
            }
            // One branch for the step, none for its updates, whose square roots then overlap: a missing one is a zero
            // gradient, which leaves sums and steps alone.  Momentum takes no such step (a decay would change its velocity,
            // and a rate of zero make NaN of an infinite one) and has no square roots: there it is left out.
            if (cnt[s]) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (MODE == kMomentumSeq && (uint32_t)u >= cnt[s]) break;
#pragma unroll
                    for (int i = 0; i < NC; ++i) item2<MODE>(w.G[i], w.acc[i], l[s].g[u][i], rp);
                }
            }
            if (PARITY) {
#pragma unroll
                for (int i = 0; i < NC; ++i) {
                    w.pe[i].x = opens ? (double)l[s].pe[i].x : w.pe[i].x;
                    w.pe[i].y = opens ? (double)l[s].pe[i].y : w.pe[i].y;
                    w.pa[i].x = opens ? (double)l[s].pa[i].x : w.pa[i].x;
                    w.pa[i].y = opens ? (double)l[s].pa[i].y : w.pa[i].y;
                }
            }
            // The set is taken in before its registers' next loads are asked for (moved up, those would go to other
            // registers and be copied at the end of the loop, which waits for them).
#pragma unroll
            for (int i = 0; i < NC; ++i) {
                asm volatile("" : "+v"(w.G[i].x), "+v"(w.G[i].y), "+v"(w.acc[i].x), "+v"(w.acc[i].y), "+v"(w.e[i].x),
                             "+v"(w.e[i].y), "+v"(w.a[i].x), "+v"(w.a[i].y) : : "memory");
                if (PARITY) asm volatile("" : "+v"(w.pe[i].x), "+v"(w.pe[i].y), "+v"(w.pa[i].x), "+v"(w.pa[i].y) : : "memory");
            }
            const uint32_t t = at[s], t1 = t + cnt[s];
            const bool took = cnt[s] != 0;
            at[s] = next;
            cnt[s] = issue_step<NC, U, PARITY>(l[s], a, col0, wkey, widx, rowheads, stripeheads, next, end);
            next += cnt[s];
            const bool last = t1 >= end;
            if (took && (last || (bool)((rowheads >> t1) & 1ull))) {          // the entry is complete
                const uint32_t x = from_lane(wkey, t);
                const rsrc_t erow = row_f32(a.E, x, D, col0), arow = row_f32(a.A, x, D, col0);
#pragma unroll
                for (int i = 0; i < NC; ++i) {
                    const D2 e64 = widen2(w.e[i]), a64 = widen2(w.a[i]);
                    finish2<MODE>(w.G[i], w.acc[i], a64, rp);
                    st2(erow, i, narrow2(D2{e64.x - w.acc[i].x, e64.y - w.acc[i].y}));
                    st2(arow, i, narrow2(w.G[i]));
                    if (PARITY) {
                        w.pe[i].x -= w.acc[i].x;
                        w.pe[i].y -= w.acc[i].y;
                        w.pa[i].x += w.G[i].x - a64.x;
                        w.pa[i].y += w.G[i].y - a64.y;
                    }
                }
                const bool closed = last || (bool)((stripeheads >> t1) & 1ull);
                if (SPLIT && PARITY && closed && from.before) {
#pragma unroll
                    for (int i = 0; i < NC; ++i) {
                        *(double2 *)(from.part + i * 128u + 2u * lane_id()) = double2{w.pe[i].x, w.pe[i].y};
                        *(double2 *)(from.part + (NC + i) * 128u + 2u * lane_id()) = double2{w.pa[i].x, w.pa[i].y};
                    }
                    from.before = false;
                } else if (PARITY && closed && !(SPLIT && last && from.goes_on)) {
                    const uint32_t g = a.geo.dk.div(x);
                    const rsrc_t perow = row_f32(a.PE, g, D, col0), parow = row_f32(a.PA, g, D, col0);
#pragma unroll
                    for (int i = 0; i < NC; ++i) {
                        st2(perow, i, narrow2(w.pe[i]));
                        st2(parow, i, narrow2(w.pa[i]));
                    }
                }
                w.clear_chain();
            }
        }
    }
}

// where the run of entry x that begins at pos ends, in the sorted list's [.., end)
__device__ __forceinline__ uint32_t run_of(const u64 *items, uint32_t pos, uint32_t end, uint32_t x)
{
    for (uint32_t q = pos;; q += kWave) {
        const uint32_t p = q + lane_id();
        const u64 other = __ballot(p >= end || item_row(items[min(p, end - 1u)]) != x);
        if (other) return q + lowest_bit(other);
    }
}

// The runs of one long stripe with fewer than `least` updates, [start, end) of a sorted list: a wave takes every
// kBucketWaves-th of them, from the w-th on, and leaves the sums of their differences in dpe and dpa.  Per run, the rows of
// the entry are asked for together with the first gradients, and the gradients of U updates are in flight while the U
// before them are applied: 8 updates per us, twice as many as the steps of the window walk, which carry the loads of rows
// that most of them do not need.
template <int NC, int MODE>
__device__ __forceinline__ void walk_runs(const RowArgs &a, const u64 *items, uint32_t start, uint32_t end, uint32_t cb,
                                          uint32_t w, uint32_t least, D2 (&dpe)[NC], D2 (&dpa)[NC])
{
    constexpr uint32_t U = NC == 1 ? 8 : 4;
    const uint32_t D = a.geo.D, lane = lane_id(), col0 = cb * NC * 128u;
    const RuleParams rp = rule_params(a.geo);
    for (uint32_t pos = start, r = 0, run_end; pos < end; pos = run_end) {
        const uint32_t x = uniform(item_row(items[pos]));
        run_end = run_of(items, pos, end, x);
        if (run_end - pos >= least || r++ % kBucketWaves != w) continue;
        const rsrc_t erow = row_f32(a.E, x, D, col0), arow = row_f32(a.A, x, D, col0);
        float2 e[NC], a0[NC], now[U][NC], next[U][NC];
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            e[i] = ld2(erow, i);
            a0[i] = ld2(arow, i);
        }
        // the gradients of updates t .. t + U - 1 (past the run's end: the last one's)
        auto load = [&](float2 (&g)[U][NC], uint32_t t) {
            const uint32_t idx = (uint32_t)items[min(t + (lane & (U - 1u)), run_end - 1u)];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                const rsrc_t grow = row_f32(a.grads, from_lane(idx, u), D, col0);
#pragma unroll
                for (int i = 0; i < NC; ++i) g[u][i] = ldg2(grow, i);
            }
        };
        load(now, pos);
        D2 G[NC], acc[NC];
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            G[i] = start2<MODE>(widen2(a0[i]));
            acc[i] = D2{0, 0};
        }
        for (uint32_t t = pos;; t += U) {
            const bool more = t + U < run_end;
            if (more) load(next, t + U);
#pragma unroll
            for (uint32_t u = 0; u < U; ++u)
                if (t + u < run_end) {
#pragma unroll
                    for (int i = 0; i < NC; ++i) item2<MODE>(G[i], acc[i], now[u][i], rp);
                }
            if (!more) break;
#pragma unroll
            for (uint32_t u = 0; u < U; ++u)
#pragma unroll
                for (int i = 0; i < NC; ++i) now[u][i] = next[u][i];
        }
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const D2 e64 = widen2(e[i]), a64 = widen2(a0[i]);
            finish2<MODE>(G[i], acc[i], a64, rp);
            st2(erow, i, narrow2(D2{e64.x - acc[i].x, e64.y - acc[i].y}));
            st2(arow, i, narrow2(G[i]));
            dpe[i].x -= acc[i].x;
            dpe[i].y -= acc[i].y;
            dpa[i].x += G[i].x - a64.x;
            dpa[i].y += G[i].y - a64.y;
        }
    }
}

// One run of many updates, [pos, end) of a sorted list, 32 columns (from col0 on) by a wave: the four groups of sixteen lanes
// take T consecutive updates each and keep their gradients in registers, exchange the updates' sums by shuffles, and apply
// the updates: 32 to a trip to memory, and no wave waits for another.  The differences are added to dpe and dpa of every lane.
// Bound by that trip: 25 updates per us, where one wave walking whole rows takes 8 (with T = 16 the same, and the registers it
// takes slow everything else down).
template <int MODE>
__device__ __forceinline__ void walk_columns(const RowArgs &a, const u64 *items, uint32_t pos, uint32_t end, uint32_t col0,
                                             D2 &dpe, D2 &dpa)
{
    constexpr uint32_t T = 8, G = 16, kStep = kWave / G * T;         // updates of a group, lanes of one, updates of a round
    constexpr bool kMomentum = MODE == kMomentumSeq;
    const uint32_t D = a.geo.D, lane = lane_id(), first = (lane / G) * T, col_lane = lane % G;
    const bool live = col0 + 2u * col_lane < D;              // D is a multiple of 4: both columns or none
    const uint32_t col = live ? col0 + 2u * col_lane : 0u, x = item_row(items[pos]);
    const RuleParams rp = rule_params(a.geo);
    float *erow = a.E + (size_t)x * D + col, *arow = a.A + (size_t)x * D + col;
    float2 g[T];
    auto load = [&](uint32_t t) {                            // past the run's end: the last update's
#pragma unroll
        for (uint32_t u = 0; u < T; ++u)
            g[u] = *(const float2 *)(a.grads + (size_t)(uint32_t)items[min(t + first + u, end - 1u)] * D + col);
    };
    load(pos);
    const float2 e = *(const float2 *)erow, a0 = *(const float2 *)arow;
    D2 state = start2<MODE>(widen2(a0)), acc = D2{0, 0};
    for (uint32_t t = pos;; t += kStep) {
        const uint32_t cnt = t + first < end ? min(T, end - t - first) : 0u;
        if (Rule<MODE>::combine) {
#pragma unroll
            for (uint32_t u = 0; u < T; ++u)
                if (u < cnt) item2<MODE>(state, acc, g[u], rp);
        } else {
            D2 s = D2{-0.0, -0.0};                           // the neutral summand
            double d = kMomentum ? decay_over(cnt, rp.mu) : 1.0;
#pragma unroll
            for (uint32_t u = 0; u < T; ++u)
                if (u < cnt) summary2<MODE>(s, g[u], rp);
            // inclusive scan over the groups of the maps v -> d * v + s, then the state before each group and after all
#pragma unroll
            for (int by = G; by < kWave; by <<= 1) {
                const double ox = __shfl_up(s.x, by, kWave), oy = __shfl_up(s.y, by, kWave);
                const double od = kMomentum ? __shfl_up(d, by, kWave) : 1.0;
                if (lane >= (uint32_t)by) {
                    s.x = kMomentum ? fma(d, ox, s.x) : s.x + ox;
                    s.y = kMomentum ? fma(d, oy, s.y) : s.y + oy;
                    if (kMomentum) d = decay(d * od, rp.mu);
                }
            }
            const double bx = __shfl_up(s.x, G, kWave), by = __shfl_up(s.y, G, kWave), bd = kMomentum ? __shfl_up(d, G, kWave) : 1.0;
            D2 mine = state;
            if (lane >= G) {
                mine.x = kMomentum ? fma(bd, state.x, bx) : state.x + bx;
                mine.y = kMomentum ? fma(bd, state.y, by) : state.y + by;
            }
            const int last = (int)(kWave - G + col_lane);
            const double lx = __shfl(s.x, last, kWave), ly = __shfl(s.y, last, kWave), ld = kMomentum ? __shfl(d, last, kWave) : 1.0;
            state.x = kMomentum ? fma(ld, state.x, lx) : state.x + lx;
            state.y = kMomentum ? fma(ld, state.y, ly) : state.y + ly;
            // the gradients are widened once more: kept in 64 bits from their sum on, they would spill
#pragma unroll
            for (uint32_t u = 0; u < T; ++u) asm volatile("" : "+v"(g[u].x), "+v"(g[u].y));
#pragma unroll
            for (uint32_t u = 0; u < T; ++u)
                if (u < cnt) item2<MODE>(mine, acc, g[u], rp);
        }
        if (t + kStep >= end) break;
        load(t + kStep);
    }
    D2 &sum = Rule<MODE>::combine ? state : acc;             // over the groups
#pragma unroll
    for (int by = G; by < kWave; by <<= 1) {
        sum.x += __shfl_xor(sum.x, by, kWave);
        sum.y += __shfl_xor(sum.y, by, kWave);
    }
    const D2 e64 = widen2(e), a64 = widen2(a0);
    finish2<MODE>(state, acc, a64, rp);
    if (live && lane < G) {
        *(float2 *)erow = narrow2(D2{e64.x - acc.x, e64.y - acc.y});
        *(float2 *)arow = narrow2(state);
    }
    dpe.x -= acc.x;
    dpe.y -= acc.y;
    dpa.x += state.x - a64.x;
    dpa.y += state.y - a64.y;
}

// A long stripe by the whole workgroup: its entries are independent, only their differences meet in the parity rows.  The waves
// share the columns of the long runs, and the short runs as a whole, and add their sums up through LDS (s_part: 6 * NC * 128
// doubles).  Every wave calls this.
// 16 384 updates on 256 rows, 256 to a stripe: 100 us a call when the owner walked it alone, 79 run by run, 58 with the runs
// shared.  With the columns of the long ones shared as well: 26 624 half Zipf 62.6 -> 55.2, 8192 half Zipf 47.7 -> 40.8, 20 000
// Zipf, k = 2, 52.9 -> 48.2, 150 000 Zipf of 256 floats 207 -> 200.
template <int NC, int MODE, bool PARITY>
__device__ __forceinline__ void walk_long_stripe(const RowArgs &a, const u64 *items, uint32_t start, uint32_t end, double *s_part)
{
    const uint32_t w = uniform(threadIdx.x / kWave), lane = lane_id(), D = a.geo.D;
    const uint32_t g = a.geo.dk.div(uniform(item_row(items[start]))), least = together(end - start);
    bool any = false;                                   // one of `least` updates: most stripes of many entries have none
    for (uint32_t q = start; q + least <= end; q += kWave) {
        const uint32_t p = min(q + lane, end - least);
        any |= __ballot(item_row(items[p]) == item_row(items[p + least - 1u])) != 0;
    }
    for (uint32_t cb = 0; cb < a.geo.ncb; ++cb) {
#pragma unroll 1
        for (int i = 0; i < NC; ++i) {
            const uint32_t col0 = (cb * NC + i) * 128u + w * 32u;
            D2 c[2] = {D2{-0.0, -0.0}, D2{-0.0, -0.0}}; // the neutral summand
            for (uint32_t pos = start, run_end; any && pos < end && col0 < D; pos = run_end) {
                run_end = run_of(items, pos, end, uniform(item_row(items[pos])));
                if (run_end - pos >= least) walk_columns<MODE>(a, items, pos, run_end, col0, c[0], c[1]);
            }
            if (lane < 16u) {
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    *(double2 *)(s_part + ((kBucketWaves + q) * NC + i) * 128u + w * 32u + 2u * lane) = double2{c[q].x, c[q].y};
            }
        }
        D2 d[2][NC];
#pragma unroll
        for (int i = 0; i < NC; ++i) d[0][i] = d[1][i] = D2{-0.0, -0.0};
        walk_runs<NC, MODE>(a, items, start, end, cb, w, least, d[0], d[1]);
        if (!PARITY) continue;
#pragma unroll
        for (uint32_t q = 0; q < 2; ++q) {              // the parity entry, by wave 0; its state, by wave 1
            const rsrc_t row = row_f32(q ? a.PA : a.PE, g, D, cb * NC * 128u);
            float2 old[NC];
#pragma unroll
            for (int i = 0; i < NC; ++i) {
                if (w == q) old[i] = ld2(row, i);
                *(double2 *)(s_part + (w * NC + i) * 128u + 2u * lane) = double2{d[q][i].x, d[q][i].y};
            }
            __syncthreads();
            if (w == q) {
#pragma unroll
                for (int i = 0; i < NC; ++i) {
                    D2 sum = widen2(old[i]);
#pragma unroll
                    for (int v = 0; v <= kBucketWaves; ++v) {
                        const int at = v < kBucketWaves ? v : kBucketWaves + q;
                        const double2 part = *(const double2 *)(s_part + (at * NC + i) * 128u + 2u * lane);
                        sum.x += part.x;
                        sum.y += part.y;
                    }
                    st2(row, i, narrow2(sum));
                }
            }
            __syncthreads();
        }
    }
}

// ================================================================================================
// a bucket's stripes, from its items in LDS
// ================================================================================================

// A list of few rows -- a hot stripe is most of a long one -- is sorted by counting: its rows, at most kFewLimit, are numbered in
// their order, and the items, which come in arrival order (`ordered`), go to the places behind those of smaller rows and of
// earlier updates of their own.  false: there are more rows, and nothing has moved.  By pieces and merging 2048 items of four
// rows take 25 us, so 5; 300 007 Zipf updates, combined, 184 -> 171 us a call.
// Lists of more than kFewLeast items: shorter ones mostly have more rows and were numbered in vain.  us a call, tried from 129 items
// on / from 193 / from 257 / from 513: 26 624 half Zipf on 2^20 rows 51.4, 51.0, 50.7, 51.0; 2^19 uniform on 2^22 rows of 16
// floats 310.2, 303.5, 303.0, 304.3; 8192 half Zipf 34.75, 34.4, 34.15, 34.45; 2^18 on 4096 rows 82.7, -, 82.2, 84.3; but 300 007 Zipf,
// combined, 174.7, 175.5, 175.4, 176.8, and 2^14 on 2520 rows, k = 63, 69.8, -, 73.0, 75.0.
constexpr uint32_t kFewLimit = 64, kFewSlots = 256, kFewLeast = 256;
struct FewRows {
    uint32_t slot[kFewSlots], number[kFewSlots];             // open addressing: row, its number
    uint32_t row[kFewLimit], at[kFewLimit], count[kBucketWaves][kFewLimit], rows;
};
static_assert(kFewLimit == kWave && kFewSlots == kBucketThreads, "a lane to a row, a thread to a slot");
__device__ __forceinline__ bool sort_few(u64 *s_item, u64 *s_tmp, uint32_t m, FewRows &t)
{
    const uint32_t tid = threadIdx.x, lane = lane_id(), w = uniform(tid / kWave);
    auto first_slot = [](uint32_t x) { return (x * 0x85EBCA77u) >> 24; };
    t.slot[tid] = kNoKey;
    t.count[w][lane] = 0;
    if (tid == 0) t.rows = 0;
    __syncthreads();
    auto *rows = (volatile __attribute__((address_space(3))) uint32_t *)&t.rows;
    for (uint32_t i = tid; i < m && *rows <= kFewLimit; i += kBucketThreads) {
        const uint32_t x = item_row(s_item[i]);
        // ends: at most kFewLimit rows are in when a thread looks, and each of the others may add one that it did not see
        for (uint32_t s = first_slot(x), tries = 0; tries < kFewSlots; s = (s + 1u) & (kFewSlots - 1u), ++tries) {
            uint32_t was = t.slot[s];
            if (was == kNoKey) {
                was = atomicCAS(&t.slot[s], kNoKey, x);
                if (was == kNoKey) atomicAdd(&t.rows, 1u);
            }
            if (was == kNoKey || was == x) break;
        }
    }
    __syncthreads();
    const uint32_t n_rows = uniform(t.rows);
    if (n_rows > kFewLimit) {
        __syncthreads();                                     // t.rows has been read
        return false;
    }
    {
        const uint32_t x = t.slot[tid];                      // numbers: the waves' rows one after the other, then by their order
        const u64 mine = __ballot(x != kNoKey);
        if (lane == 0) t.at[w] = (uint32_t)__popcll(mine);
        __syncthreads();
        uint32_t at = (uint32_t)__popcll(mine & bits_below(lane));
        for (uint32_t v = 0; v < w; ++v) at += t.at[v];
        if (x != kNoKey) t.row[at] = x;
        __syncthreads();
        uint32_t number = 0;
        for (uint32_t i = 0; i < n_rows; ++i) number += t.row[i] < x ? 1u : 0u;
        t.number[tid] = number;
        __syncthreads();
    }
    auto number_of = [&](uint32_t x) {
        uint32_t s = first_slot(x);
        while (t.slot[s] != x) s = (s + 1u) & (kFewSlots - 1u);
        return t.number[s];
    };
    // every wave a contiguous part of the list, 64 at a time: the lanes of one row, and how many of them are before a lane
    const uint32_t part = (m + kBucketThreads - 1) / kBucketThreads * kWave, lo = min(w * part, m), hi = min(lo + part, m);
    auto peers_of = [&](bool in, uint32_t number) {
        u64 peers = __ballot(in);
#pragma unroll
        for (int b = 0; b < 6; ++b) {
            const bool bit = (number >> b) & 1u;
            const u64 bal = __ballot(bit);
            peers &= bit ? bal : ~bal;
        }
        return peers;
    };
    for (uint32_t i0 = lo; i0 < hi; i0 += kWave) {
        const bool in = i0 + lane < hi;
        const uint32_t number = in ? number_of(item_row(s_item[i0 + lane])) : 0u;
        const u64 peers = peers_of(in, number);
        if (in && (peers & bits_below(lane)) == 0) t.count[w][number] += (uint32_t)__popcll(peers);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    if (w == 0) {                                            // lane: a row; where each wave's updates of it begin
        uint32_t cnt[kBucketWaves], all = 0;
#pragma unroll
        for (int v = 0; v < kBucketWaves; ++v) {
            cnt[v] = t.count[v][lane];
            all += cnt[v];
        }
        uint32_t incl = all;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const uint32_t up = __shfl_up(incl, d, kWave);
            if (lane >= (uint32_t)d) incl += up;
        }
        uint32_t at = incl - all;
#pragma unroll
        for (int v = 0; v < kBucketWaves; ++v) {
            t.count[v][lane] = at;
            at += cnt[v];
        }
    }
    __syncthreads();
    for (uint32_t i0 = lo; i0 < hi; i0 += kWave) {
        const bool in = i0 + lane < hi;
        const u64 it = in ? s_item[i0 + lane] : 0ull;
        const uint32_t number = in ? number_of(item_row(it)) : 0u;
        const u64 peers = peers_of(in, number);
        const uint32_t at = t.count[w][number], below = (uint32_t)__popcll(peers & bits_below(lane));
        __builtin_amdgcn_wave_barrier();
        if (in) {
            s_tmp[at + below] = it;
            if (below == 0) t.count[w][number] = at + (uint32_t)__popcll(peers);
        }
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    for (uint32_t i = tid; i < m; i += kBucketThreads) s_item[i] = s_tmp[i];
    __syncthreads();
    return true;
}

// Sorts m distinct items, with room for as many, and for 128 at least, in tmp (both to whole pieces of 64).  Up to 128: the waves
// count for each item the smaller ones of a part of the list, which is its place.  More: every wave orders pieces of 64 in the
// same way -- reads that all lanes share --, an item looks up its place in the other pieces of its eight by binary search, and
// lists of eight and more pieces are merged two and two.  Bound by the latency of LDS.  us a call when every item looked itself up
// in all other pieces, and only 64 were counted by one wave / so: 2048 uniform updates 16.9 / 16.2, 26 624 half Zipf 48.2 / 47.6,
// 300 007 Zipf, combined, where 1250 items took 30 us, 187.5 / 184.8; merged from 64 on, 65 536 half Zipf 84.9, so 82.9.  Short
// loops: code that only a few long lists run through costs more in instruction fetches than it saves.
__device__ __forceinline__ void sort_items(u64 *s_item, u64 *s_tmp, uint32_t m, bool ordered, FewRows &few, uint32_t few_least = kFewLeast)
{
    const uint32_t tid = threadIdx.x, lane = lane_id(), w = uniform(tid / kWave);
    const uint32_t pieces = (m + kWave - 1) / kWave;
    if (pieces <= 2u) {
        const uint32_t width = pieces * kWave, at = tid % width, share = pieces * pieces * (kWave / kBucketWaves);
        uint32_t *part = (uint32_t *)s_tmp;
        const u64 it = at < m ? s_item[at] : ~0ull;
        const uint32_t lo = (w / pieces) * share, hi = min(lo + share, m);
        uint32_t rank = 0;
#pragma unroll 8
        for (uint32_t j = lo; j < hi; ++j) rank += s_item[j] < it ? 1u : 0u;
        part[tid] = rank;
        __syncthreads();
        if (tid < m) {
            rank = 0;
            for (uint32_t from = tid; from < (uint32_t)kBucketThreads; from += width) rank += part[from];
            s_item[rank] = it;
        }
        __syncthreads();
        return;
    }
    if (__builtin_expect(ordered && m > few_least, 0) && sort_few(s_item, s_tmp, m, few)) return;
    if (tid < pieces * kWave - m) s_item[m + tid] = ~0ull;       // fewer than 64: what is read behind the list counts as larger
    __syncthreads();
    for (uint32_t i = tid; i - lane < m; i += kBucketThreads) {
        const u64 it = s_item[i], *piece = s_item + (i - lane);
        uint32_t rank = 0;
#pragma unroll 8
        for (uint32_t j = 0; j < (uint32_t)kWave; j += 2) {
            const ulonglong2 v = *(const ulonglong2 *)(piece + j);
            rank += (v.x < it ? 1u : 0u) + (v.y < it ? 1u : 0u);
        }
        if (i < m) s_tmp[i - lane + rank] = it;
        else s_tmp[i] = ~0ull;                                   // the padding stays behind the list
    }
    __syncthreads();
    constexpr uint32_t kGroup = 8;                               // pieces that are merged at once
    for (uint32_t i = tid; i < m; i += kBucketThreads) {
        const u64 it = s_tmp[i];
        const uint32_t own = i / kWave, first = own & ~(kGroup - 1u), last = min(first + kGroup, pieces);
        uint32_t rank = lane;                                    // its place in its own piece
        for (uint32_t o = first; o < last; o += 2) {             // two other pieces at a time
            const u64 *pa = s_tmp + o * kWave, *pb = pa + (o + 1 < last ? kWave : 0);
            uint32_t la = 0, lb = 0;
#pragma unroll
            for (uint32_t step = kWave; step > 0; step /= 2) {
                const uint32_t ta = la + step, tb = lb + step;
                const u64 va = pa[min(ta, (uint32_t)kWave) - 1u], vb = pb[min(tb, (uint32_t)kWave) - 1u];
                la = ta <= (uint32_t)kWave && va < it ? ta : la;
                lb = tb <= (uint32_t)kWave && vb < it ? tb : lb;
            }
            rank += (o != own ? la : 0u) + (o + 1 < last && o + 1 != own ? lb : 0u);
        }
        s_item[first * kWave + rank] = it;
    }
    __syncthreads();
    u64 *src = s_item, *dst = s_tmp;
    for (uint32_t len = kGroup * kWave; len < m; len *= 2) {
        constexpr uint32_t U = 2;                                // items of a thread at a time
        for (uint32_t i0 = tid; i0 < m; i0 += U * kBucketThreads) {
            u64 it[U];
            uint32_t mate[U], size[U], rank[U];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                const uint32_t i = min(i0 + u * kBucketThreads, m - 1u);
                it[u] = src[i];
                mate[u] = (i & ~(2u * len - 1u)) + (i & len ? 0u : len);
                size[u] = mate[u] < m ? min(len, m - mate[u]) : 0u;
                mate[u] = size[u] ? mate[u] : 1u;                // no other list: nothing behind this one is read
                rank[u] = 0;
            }
            for (uint32_t step = len; step > 0; step /= 2) {
#pragma unroll
                for (uint32_t u = 0; u < U; ++u) {
                    const uint32_t t = rank[u] + step;
                    const u64 v = src[mate[u] + min(t, size[u]) - 1u];
                    rank[u] = t <= size[u] && v < it[u] ? t : rank[u];
                }
            }
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                const uint32_t i = i0 + u * kBucketThreads;
                if (i < m) dst[(i & ~len) + rank[u]] = it[u];
            }
        }
        __syncthreads();
        u64 *const sorted = dst;
        dst = src;
        src = sorted;
    }
    if (src == s_item) return;
    for (uint32_t i = tid; i < m; i += kBucketThreads) s_item[i] = src[i];
    __syncthreads();
}

template <uint32_t CAP>
struct ListShared {
    // stripes for other workgroups, and those that the whole workgroup walks: start | end << 16
    uint32_t heavy[CAP / (kWave - kBucketChunk)], longs[CAP / (kWave - kBucketChunk)];
    uint32_t n_heavy, n_long, chunk;
    uint32_t handed[kBucketWaves];           // of a wave's part of a list that is cut at entries (kNothing, ...)
    uint32_t srv[2 * kBucketMaxServers];
};

// Cuts a list of m items, at most kSplitWords * 64, into a part for each wave, at entries, with equally many steps of up to U updates
// of an entry to a part.  false: a part does not fit a window -- or, where a stripe may be too long for a window, has a run that the
// workgroup had better share, which is what limits such a list to a part of kTogether for each wave.  The same for every wave.
constexpr uint32_t kSplitWords = 2, kSplitLeast = 16;
static_assert(kSplitWords * kWave == kBucketWaves * kTogether, "longer lists are never cut");
template <uint32_t U>
__device__ __forceinline__ bool split_list(const u64 *items, uint32_t m, uint32_t (&bound)[kBucketWaves + 1])
{
    const uint32_t lane = lane_id();
    u64 heads[kSplitWords];
    uint32_t before[kSplitWords], begin = 0, all = 0;        // begin: of the entry that goes on into the word
#pragma unroll
    for (uint32_t j = 0; j < kSplitWords; ++j) {
        heads[j] = 0;
        before[j] = all;
        if (j * kWave >= m) continue;
        const uint32_t p = j * kWave + lane, q = min(p, m - 1u);
        heads[j] = __ballot(p < m && (p == 0 || item_row(items[q]) != item_row(items[max(q, 1u) - 1u])));
        const u64 mine = heads[j] & bits_below(lane + 1u);
        const uint32_t from = mine ? j * kWave + 63u - (uint32_t)__builtin_clzll(mine) : begin;
        const u64 steps = __ballot(p < m && (p - from) % U == 0);
        before[j] += (uint32_t)__popcll(steps & bits_below(lane));
        all += (uint32_t)__popcll(steps);
        if (heads[j]) begin = j * kWave + 63u - (uint32_t)__builtin_clzll(heads[j]);
    }
    const uint32_t most = m <= (uint32_t)kWave ? kWave - 1u : kTogether;
    bound[0] = 0;
    bool fits = true;
#pragma unroll
    for (uint32_t v = 1; v <= (uint32_t)kBucketWaves; ++v) {
        uint32_t at = m;
#pragma unroll
        for (int j = kSplitWords - 1; j >= 0 && v < (uint32_t)kBucketWaves; --j) {
            const u64 reached = heads[j] & __ballot(before[j] * kBucketWaves >= v * all);
            if (reached) at = j * kWave + lowest_bit(reached);
        }
        bound[v] = at;
        fits = fits && at - bound[v - 1u] <= most;
    }
    return fits;
}

// Which lists that is tried on: of few stripes, more than a wave's and fewer than kSplitStripes.  Where one is longer than a window
// and entries have several updates, what the whole workgroup walks is faster as it is (144 298 uniform updates, combined, 92 to a
// stripe of ten entries of 512 floats, 133 us, cut 159; 20 301 on 856 rows of 64 floats 28.7, 31.1; but 466 158, combined, 72 to a stripe of
// 63 entries, 281, cut 272).
__device__ __forceinline__ bool few_stripes(const u64 *items, uint32_t m, const Divider &dk)
{
    if (m <= kSplitLeast || m > kSplitWords * kWave) return false;
    uint32_t stripes = 0, entries = 0;
    bool longer = false;
    for (uint32_t p0 = 0; p0 < m; p0 += kWave) {
        const uint32_t p = p0 + lane_id(), q = min(p, m - 1u), x = item_row(items[q]), g = dk.div(x), left = item_row(items[max(q, 1u) - 1u]);
        entries += (uint32_t)__popcll(__ballot(p < m && (p == 0 || x != left)));
        stripes += (uint32_t)__popcll(__ballot(p < m && (p == 0 || g != dk.div(left))));
        longer |= __ballot(p + kWave < m && g == dk.div(item_row(items[min(p + kWave, m - 1u)]))) != 0;
    }
    return stripes < kSplitStripes && !(longer && 3u * entries < m);
}

// Applies a list of few stripes in parts of equal length, a wave to each, if it can be cut into such; false: nothing has been done.
// Where a stripe goes from one part to the next its parity rows are put together afterwards by the wave that has opened it.
// s_part: 6 * NC * 128 doubles.  A stripe a wave, 64 updates of four stripes kept the waves busy from 1.5 to 12 us: 65 536
// uniform updates on 2^14 rows 40.5 us a call, so 36.5, of 256 floats 66.4, now 59.1; on 1024 rows 46.8, 46.1.  Lists of many
// stripes, whose waves come out even by themselves, would lose (8192 half Zipf on 2^16 rows 34.9, all lists cut 36.3), and what the
// kernel takes for it costs the others up to 1 % (65 536 Zipf on 2^16 rows 72.2, 73.0; 12 000 on 2^14 40.9, 41.6).
// What a part begins with: a stripe of its own, the end of an earlier part's, or one that takes all of it.
enum { kNothing, kSome, kAll, kEmpty };
template <int NC, int MODE, bool PARITY, int Q, int U>
__device__ __forceinline__ bool apply_split(const RowArgs &a, const u64 *items, uint32_t m, uint32_t *handed, double *s_part)
{
    const uint32_t lane = lane_id(), w = uniform(threadIdx.x / kWave);
    const Divider dk = a.geo.dk;
    if (!few_stripes(items, m, dk)) return false;
    uint32_t bound[kBucketWaves + 1];
    if (!split_list<U>(items, m, bound)) return false;
    uint32_t p0 = bound[0], out = bound[1];
#pragma unroll
    for (uint32_t v = 1; v < (uint32_t)kBucketWaves; ++v)
        if (w == v) p0 = bound[v], out = bound[v + 1u];
    const uint32_t end = out - p0;
    const u64 it = p0 + lane < m ? items[p0 + lane] : ~0ull;
    const uint32_t wkey = item_row(it), widx = (uint32_t)it;
    uint32_t leftk = __shfl_up(wkey, 1, kWave);
    if (lane == 0) leftk = p0 ? item_row(items[p0 - 1]) : kNoKey;
    const bool valid = wkey != kNoKey;
    const u64 rowheads = __ballot(!valid || leftk == kNoKey || leftk != wkey);
    const u64 stripeheads = __ballot(valid && (leftk == kNoKey || dk.div(leftk) != dk.div(wkey)));
    const u64 opened = stripeheads & bits_below(end);
    const bool before = end && !(stripeheads & 1ull), goes_on = out < m && !((stripeheads >> end) & 1ull);
    if (lane == 0) handed[w] = end == 0 ? kEmpty : !before ? kNothing : opened ? kSome : kAll;
    for (uint32_t cb = 0; cb < a.geo.ncb; ++cb) {
        Walk<NC> walk;
        if (end)                                             // the first wave begins with a stripe
            walk_window<NC, MODE, PARITY, Q, U, true>(a, wkey, widx, rowheads, stripeheads, 0, end, cb, walk,
                                                      Shared{before, goes_on, s_part + (w - 1u) * 2u * NC * 128u});
        __syncthreads();
        if (PARITY && goes_on && opened) {
            for (uint32_t v = w + 1u; v < (uint32_t)kBucketWaves; ++v) {
                const uint32_t what = uniform(handed[v]);
                if (what == kEmpty) continue;
                if (what == kNothing) break;
                const double *from = s_part + (v - 1u) * 2u * NC * 128u;
#pragma unroll
                for (int i = 0; i < NC; ++i) {
                    const double2 pe = *(const double2 *)(from + i * 128u + 2u * lane), pa = *(const double2 *)(from + (NC + i) * 128u + 2u * lane);
                    walk.pe[i].x += pe.x;
                    walk.pe[i].y += pe.y;
                    walk.pa[i].x += pa.x;
                    walk.pa[i].y += pa.y;
                }
                if (what == kSome) break;
            }
            const uint32_t g = dk.div(from_lane(wkey, end - 1u)), col0 = cb * NC * 128u;
            const rsrc_t perow = row_f32(a.PE, g, a.geo.D, col0), parow = row_f32(a.PA, g, a.geo.D, col0);
#pragma unroll
            for (int i = 0; i < NC; ++i) {
                st2(perow, i, narrow2(walk.pe[i]));
                st2(parow, i, narrow2(walk.pa[i]));
            }
        }
        __syncthreads();                                     // the parts have been read: the caller may have other uses for them
    }
    return true;
}

// Applies every stripe of a sorted list of m items (m <= CAP).  A list of few stripes is cut at entries (apply_split;
// CUT).  Of others chunks of a few positions are handed to the waves as they come free; a wave owns the stripes that open in its
// chunk.  A stripe that does not end inside the wave's 64-position window
//   - is only listed in sh.heavy if it has a run of heavy_run updates and that makes up more than half of it, or it has
//     shared_stripe updates (RUNS; otherwise: if it has shared_stripe updates);
//   - is walked by the whole workgroup afterwards otherwise (s_part: room for walk_long_stripe).
// A barrier has to lie between the last write of the list and this call; the call ends with one.
template <int NC, int MODE, bool PARITY, bool RUNS, bool CUT, uint32_t CAP>
__device__ __forceinline__ void apply_list(const RowArgs &a, const u64 *items, uint32_t m, uint32_t heavy_run,
                                           uint32_t shared_stripe, ListShared<CAP> &sh, double *s_part)
{
    constexpr int kQ = 2, kU = NC == 1 ? 4 : 2;
    const uint32_t lane = lane_id();
    const Divider dk = a.geo.dk;
    if (threadIdx.x == 0) {
        sh.n_heavy = sh.n_long = 0;
        sh.chunk = kBucketWaves;
    }
    __syncthreads();
    if (CUT && apply_split<NC, MODE, PARITY, kQ, kU>(a, items, m, sh.handed, s_part)) return;
    // a chunk for each wave of a short list
    const uint32_t CH = min(kBucketChunk, max(1u, (m + kBucketWaves - 1u) / kBucketWaves));
    for (uint32_t c = uniform(threadIdx.x / kWave); c * CH < m;) {
        const uint32_t p0 = c * CH;
        if (lane == 0) c = atomicAdd(&sh.chunk, 1u);         // the chunk after this one
        c = uniform(c);
        const u64 it = p0 + lane < m ? items[p0 + lane] : ~0ull;
        const uint32_t wkey = item_row(it), widx = (uint32_t)it;
        uint32_t leftk = __shfl_up(wkey, 1, kWave);
        if (lane == 0) leftk = p0 ? item_row(items[p0 - 1]) : kNoKey;
        const bool valid = wkey != kNoKey;
        const u64 rowheads = __ballot(!valid || leftk == kNoKey || leftk != wkey);
        const u64 stripeheads = __ballot(valid && (leftk == kNoKey || dk.div(leftk) != dk.div(wkey)));
        const u64 owned = stripeheads & bits_below(CH);
        if (!owned) continue;
        const uint32_t first = lowest_bit(owned), last = 63u - (uint32_t)__builtin_clzll(owned);
        const u64 after = stripeheads & ~bits_below(last + 1);
        const bool inside = after != 0ull || p0 + kWave >= m;
        const uint32_t end = inside ? (after ? lowest_bit(after) : min((uint32_t)kWave, m - p0)) : last;
        // the stripe that goes on behind the window: where it ends, and how long its runs are
        const uint32_t big_start = p0 + last;
        uint32_t big_end = big_start;
        if (!inside) {
            const uint32_t g = dk.div(from_lane(wkey, last));
            bool long_run = false, one_run = false;                 // of heavy_run updates; of more than half of the stripe
            for (;;) {
                const uint32_t p = big_end + lane;
                const uint32_t key = p < m ? item_row(items[p]) : kNoKey;
                const bool same = key != kNoKey && dk.div(key) == g;
                if (RUNS && __ballot(same && p + heavy_run - 1 < m && item_row(items[min(p + heavy_run - 1, m - 1)]) == key)) long_run = true;
                const u64 other = __ballot(!same);
                if (other) {
                    big_end += lowest_bit(other);
                    break;
                }
                big_end += kWave;
            }
            const uint32_t size = big_end - big_start, half = size / 2u;
            for (uint32_t q = big_start; long_run && q + half < big_end; q += kWave) {
                const uint32_t p = min(q + lane, big_end - half - 1u);
                if (__ballot(item_row(items[p + half]) == item_row(items[p]))) one_run = true;
            }
            const uint32_t what = big_start | (big_end << 16);
            if (lane == 0) {
                if ((!RUNS || long_run) && (one_run || size >= shared_stripe)) sh.heavy[atomicAdd(&sh.n_heavy, 1u)] = what;
                else sh.longs[atomicAdd(&sh.n_long, 1u)] = what;
            }
        }
        if (first < end)
            for (uint32_t cb = 0; cb < a.geo.ncb; ++cb) {
                Walk<NC> walk;
                walk_window<NC, MODE, PARITY, kQ, kU, false>(a, wkey, widx, rowheads, stripeheads, first, end, cb, walk, Shared{});
            }
    }
    __syncthreads();
    const uint32_t n_long = uniform(sh.n_long);
    for (uint32_t i = 0; i < n_long; ++i) {                  // their order in the list may vary; they share nothing
        const uint32_t what = uniform(sh.longs[i]);
        walk_long_stripe<NC, MODE, PARITY>(a, items, what & 0xFFFFu, what >> 16, s_part);
    }
    if (n_long) __syncthreads();
}

// Combined rules: one entry update and one parity update per modified entry (Sec. 3.6, Sec. 4.4).  The list is sorted.
__device__ __forceinline__ void count_list(const Geometry &geo, const u64 *items, uint32_t m, uint32_t *s_srv,
                                           u64 *load_data, u64 *load_parity)
{
    const uint32_t S = geo.S;
    for (uint32_t i = threadIdx.x; i < 2 * S; i += kBucketThreads) s_srv[i] = 0;
    __syncthreads();
    for (uint32_t p = threadIdx.x; p < m; p += kBucketThreads) {
        const uint32_t x = item_row(items[p]);
        if (p && item_row(items[p - 1]) == x) continue;
        const uint32_t g = geo.dk.div(x), j = x - g * geo.k;
        atomicAdd(&s_srv[geo.dS.mod(g + 1 + j)], 1u);
        atomicAdd(&s_srv[S + geo.dS.mod(g)], 1u);
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < 2 * S; i += kBucketThreads) {
        u64 *to = i < S ? load_data : load_parity;
        if (s_srv[i] && to) atomicAdd(&to[i < S ? i : i - S], (u64)s_srv[i]);
    }
    __syncthreads();
}

// The header of a call through the kernels of small batches (one thread; no other workgroup of the launch touches it).
__device__ __forceinline__ void begin_batch(Header *h, uint32_t n, bool clear_sticky)
{
    if (clear_sticky) {
        h->err_sticky = 0;
        h->buf_count = 0;
        h->free_count = 0;
        h->bump = 0;
    }
    h->batch_bad = 0;
    h->n_long = 0;
    h->n_pieces = 0;
    h->n_long_items = 0;
    h->n_batch = n;
    h->n_valid = n;
    h->n_held = 0;
    h->n_heavy = 0;
    h->n_segments = 0;
    h->heavy_ticket = 0;
    for (uint32_t c = 0; c < kMidClasses; ++c) h->n_mid[c] = 0;
}

// the runs of a sorted list, by the workgroup: every wave its part (s_sum: kBucketWaves * 4); ends with a barrier
__device__ __forceinline__ DirectList count_runs(const u64 *items, uint32_t m, uint32_t *s_sum)
{
    const uint32_t w = uniform(threadIdx.x / kWave), third = m / 3u;
    uint32_t sum[4] = {0, 0, 0, 0};
    for (uint32_t q = w * kWave; q < m; q += kBucketThreads) {
        const uint32_t p = min(q + lane_id(), m - 1u), x = item_row(items[p]);
        const bool in = q + lane_id() < m, head = in && (p == 0 || item_row(items[p - 1u]) != x);
        auto goes_on = [&](uint32_t updates) { return in && p + updates <= m && item_row(items[min(p + updates, m) - 1u]) == x; };
        const u64 heads = __ballot(head), longer = __ballot(goes_on(kDirectRun));
        sum[0] += (uint32_t)__popcll(heads);
        sum[1] += (uint32_t)__popcll(heads & longer);
        sum[2] += (uint32_t)__popcll(longer);
        sum[3] |= __ballot(goes_on(third)) ? 1u : 0u;
    }
    if (lane_id() == 0)
#pragma unroll
        for (int i = 0; i < 4; ++i) s_sum[w * 4 + i] = sum[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        sum[i] = 0;
#pragma unroll
        for (int v = 0; v < kBucketWaves; ++v) sum[i] += s_sum[v * 4 + i];
        sum[i] = uniform(sum[i]);
    }
    __syncthreads();
    // a run of r updates goes on for kDirectRun from r - kDirectRun + 1 of its positions
    return DirectList{m, sum[0], sum[1], m - (sum[2] + sum[1] * (kDirectRun - 1u)), sum[3] != 0};
}

// 2 G columns of one stripe, [start, end) of a sorted list, by a workgroup: as in long_runs.h, with T updates to a group of G lanes:
// 256 updates to a round with G = 8, 512 with G = 4.  A run of fewer than kGroupRun updates goes to one group, all of them at once
// behind the long ones: each took a round by itself.  ex: both halves free; ends with a barrier.
constexpr uint32_t kGroupRun = kDirectRun;
template <int MODE, bool PARITY, int G>
__device__ __forceinline__ void stripe_columns(const RowArgs &a, const u64 *items, uint32_t start, uint32_t end, uint32_t cg,
                                               ExchangeOf<kBucketWaves, G> (&ex)[2])
{
    constexpr int T = 8;
    constexpr uint32_t kGroups = kBucketThreads / G, kRound = kGroups * T;
    const uint32_t D = a.geo.D, tid = threadIdx.x, lane = lane_id(), w = uniform(tid / kWave);
    const uint32_t col_lane = lane % G, sub = tid / G, col = (cg * G + col_lane) * 2u;
    const bool live = col < D;                                      // D is a multiple of 4: both columns or none
    const RuleParams rp = rule_params(a.geo);
    const uint32_t g = a.geo.dk.div(uniform(item_row(items[start])));
    D2 pe = D2{-0.0, -0.0}, pa = D2{-0.0, -0.0};                    // a group's differences; the neutral summand
    uint32_t buf = 0, runs = 0, own0 = start, len0 = 0, own1 = start, len1 = 0;       // the group's runs: a stripe has 64 at most
    // the gradients of updates r0 + off .. of the run at pos, zeros past its end
    auto rows = [&](float2 (&r)[T], uint32_t pos, uint32_t off, uint32_t L) {
        uint32_t mine[T / G];
#pragma unroll
        for (int q = 0; q < T / G; ++q) mine[q] = (uint32_t)items[pos + min(off + q * G + col_lane, L - 1u)];
#pragma unroll
        for (int u = 0; u < T; ++u) {
            const uint32_t i = __shfl(mine[u / G], (int)(lane - col_lane + u % G), kWave);
            r[u] = float2{0, 0};
            if (live && off + u < L) r[u] = *(const float2 *)(a.grads + (size_t)i * D + col);
        }
    };
    auto store = [&](uint32_t x, D2 state, D2 acc, const D2 &a64, bool mine) {
        finish2<MODE>(state, acc, a64, rp);
        if (!mine) return;
        float2 *e = (float2 *)(a.E + (size_t)x * D + col);
        const D2 e64 = widen2(*e);
        *e = narrow2(D2{e64.x - acc.x, e64.y - acc.y});
        *(float2 *)(a.A + (size_t)x * D + col) = narrow2(state);
        pe.x -= acc.x;
        pe.y -= acc.y;
        pa.x += state.x - a64.x;
        pa.y += state.y - a64.y;
    };
    for (uint32_t pos = start, run_end; pos < end; pos = run_end) {
        const uint32_t x = uniform(item_row(items[pos]));
        run_end = run_of(items, pos, end, x);
        const uint32_t L = run_end - pos;
        if (L < kGroupRun) {
            if (runs == sub) own0 = pos, len0 = L;
            if (runs == sub + kGroups) own1 = pos, len1 = L;
            ++runs;
            continue;
        }
        float2 gr[T], nx[T];
        rows(nx, pos, sub * T, L);
        D2 a64 = D2{0, 0};
        if (live) a64 = widen2(*(const float2 *)(a.A + (size_t)x * D + col));
        D2 state = start2<MODE>(a64), acc = D2{0, 0};
        for (uint32_t r0 = 0; r0 < L; r0 += kRound) {
            const uint32_t off = r0 + sub * T, cnt = off < L ? min((uint32_t)T, L - off) : 0u;
#pragma unroll
            for (int u = 0; u < T; ++u) gr[u] = nx[u];
            if (r0 + kRound < L) rows(nx, pos, off + kRound, L);
            if (Rule<MODE>::combine) {                              // a sum: nothing to exchange before the run's end
#pragma unroll
                for (int u = 0; u < T; ++u) {                       // zeros past the end of the run
                    acc.x += (double)gr[u].x;
                    acc.y += (double)gr[u].y;
                }
                continue;
            }
            double ed;
            const D2 before = heavy_sums<MODE>(gr, cnt, rp, ex[buf], w, ed);
            __syncthreads();
            D2 mine = heavy_fold<MODE>(state, ex[buf], w, before, ed);
#pragma unroll
            for (int u = 0; u < T; ++u) asm volatile("" : "+v"(gr[u].x), "+v"(gr[u].y));     // widened once more (walk_columns)
#pragma unroll
            for (int u = 0; u < T; ++u) {
                if ((uint32_t)u < cnt) item2<MODE>(mine, acc, gr[u], rp);
            }
            buf ^= 1u;                                              // a half is written again only behind the other's barrier
        }
        acc = heavy_total(acc, ex[buf], w);
        buf ^= 1u;
        if (Rule<MODE>::combine) {
            state = acc;
            acc = D2{0, 0};
        }
        store(x, state, acc, a64, live && sub == 0);
    }
    for (uint32_t half = 0; half < runs; half += kGroups) {         // once or twice
        const uint32_t pos = half ? own1 : own0, L = half ? len1 : len0, x = item_row(items[pos]);
        uint32_t most = L;
#pragma unroll
        for (int by = G; by < kWave; by <<= 1) most = max(most, __shfl_xor(most, by, kWave));
        D2 a64 = D2{0, 0};
        if (live && L) a64 = widen2(*(const float2 *)(a.A + (size_t)x * D + col));
        D2 state = start2<MODE>(a64), acc = D2{0, 0};
        for (uint32_t r0 = 0; r0 < most; r0 += T) {
            float2 gr[T];
            rows(gr, pos, r0, max(L, 1u));
#pragma unroll
            for (int u = 0; u < T; ++u) {
                if (r0 + u < L) item2<MODE>(state, acc, gr[u], rp);
            }
        }
        store(x, state, acc, a64, live && L);
    }
    if (PARITY) {
        __syncthreads();                                            // ex has been read
        // over the groups, in their order; the first group's lanes add the sums up
#pragma unroll
        for (int by = G; by < kWave; by <<= 1) {
            pe.x += __shfl_xor(pe.x, by, kWave);
            pe.y += __shfl_xor(pe.y, by, kWave);
            pa.x += __shfl_xor(pa.x, by, kWave);
            pa.y += __shfl_xor(pa.y, by, kWave);
        }
        if (lane < (uint32_t)G) {
            ex[0].sum[w][col_lane][0] = pe.x;
            ex[0].sum[w][col_lane][1] = pe.y;
            ex[1].sum[w][col_lane][0] = pa.x;
            ex[1].sum[w][col_lane][1] = pa.y;
        }
        __syncthreads();
        if (live && sub == 0) {
            float2 *to = (float2 *)(a.PE + (size_t)g * D + col), *to_state = (float2 *)(a.PA + (size_t)g * D + col);
            D2 pe64 = widen2(*to), pa64 = widen2(*to_state);
#pragma unroll
            for (int v = 0; v < kBucketWaves; ++v) {
                pe64.x += ex[0].sum[v][col_lane][0];
                pe64.y += ex[0].sum[v][col_lane][1];
                pa64.x += ex[1].sum[v][col_lane][0];
                pa64.y += ex[1].sum[v][col_lane][1];
            }
            *to = narrow2(pe64);
            *to_state = narrow2(pa64);
        }
    }
    __syncthreads();
}

}  // namespace ecrm
