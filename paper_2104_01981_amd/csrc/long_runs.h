// A long run of updates of one entry by a workgroup, 16 columns at a time: the columns of a row are independent chains, so
// a run spreads over D / 16 workgroups that never wait for each other and read every gradient once (64-byte pieces).  A
// lane holds two columns of kHeavyT consecutive updates; the 64 groups of eight lanes exchange their summaries by shuffles
// and, across waves, through LDS, and take their steps from registers: 1024 updates per round.  Shared by heavy_stripes
// (buckets.hip) and the reads during a recovery (reads.hip).
#pragma once

#include "rows.h"

namespace ecrm {

constexpr uint32_t kHeavyCols = 16;          // columns of a job
constexpr int kHeavyThreads = 512;
constexpr int kHeavyWaves = kHeavyThreads / kWave;
constexpr int kHeavyT = 16;                  // updates that a group of eight lanes takes at a time

// The decay over a number of updates, a power of mu.  One that underflows is kept at the smallest normal number unless mu
// itself is zero: a decay of zero would make NaN of an infinite velocity, which the rule keeps infinite.  What it adds to
// a finite one is below 1e-269, nothing in 32 bits.
__device__ __forceinline__ double decay(double power, double mu) { return mu > 0.0 ? fmax(power, 2.2250738585072014e-308) : power; }

// the decay over m updates
__device__ __forceinline__ double decay_over(uint32_t m, double mu)
{
    double r = 1.0, p = mu;
    for (; m; m >>= 1) {
        if (m & 1u) r = decay(r * p, mu);
        p = decay(p * p, mu);
    }
    return r;
}

// gradient rows of a run's updates at, at + 1 (past its end: its last update's)
template <typename I>
__device__ __forceinline__ void heavy_indices(const I *run, uint32_t L, uint32_t at, uint32_t &i0, uint32_t &i1)
{
    i0 = (uint32_t)run[min(at, L - 1u)];
    i1 = (uint32_t)run[min(at + 1u, L - 1u)];
}

// two columns of the run's updates at .. at + T - 1, zeros past its end
template <int T>
__device__ __forceinline__ void heavy_rows(float2 (&r)[T], const float *grads, uint32_t D, uint32_t col, bool live, uint32_t i0,
                                           uint32_t i1, uint32_t lane, uint32_t at, uint32_t L)
{
#pragma unroll
    for (int u = 0; u < T; ++u) {
        const uint32_t idx = __shfl(u & 1 ? i1 : i0, (int)((lane & 56u) + u / 2), kWave);
        r[u] = float2{0, 0};
        if (live && at + u < L) r[u] = *(const float2 *)(grads + (size_t)idx * D + col);
    }
}

// what the waves exchange: sums (or, at the end of a run, steps) of two columns a lane, and the decay over a wave's updates.  G:
// lanes of a group.
template <int WAVES, int G = 8>
struct ExchangeOf {
    double sum[WAVES][G][2], dec[WAVES];
};
using HeavyExchange = ExchangeOf<kHeavyWaves>;
// Sums of a round: every wave leaves that of its updates in ex; returned is what lies before the lane's group inside its
// wave, with its decay.
template <int MODE, int T, int WAVES, int G>
__device__ __forceinline__ D2 heavy_sums(const float2 (&gr)[T], uint32_t cnt, const RuleParams &rp, ExchangeOf<WAVES, G> &ex,
                                         uint32_t w, double &before_decay)
{
    constexpr bool kMomentum = MODE == kMomentumSeq;
    const uint32_t lane = lane_id(), col_lane = lane % G;
    D2 s = D2{-0.0, -0.0};                              // the neutral summand: +0.0 would take a -0.0's sign
    double d = kMomentum ? decay_over(cnt, rp.mu) : 1.0;
#pragma unroll
    for (int u = 0; u < T; ++u) {
        if ((uint32_t)u < cnt) summary2<MODE>(s, gr[u], rp);
    }
    // inclusive scan over the wave's groups of the maps v -> d * v + s
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
    if (lane >= (uint32_t)(kWave - G)) {
        ex.sum[w][col_lane][0] = s.x;
        ex.sum[w][col_lane][1] = s.y;
        if (col_lane == 0) ex.dec[w] = d;
    }
    D2 before = D2{__shfl_up(s.x, G, kWave), __shfl_up(s.y, G, kWave)};
    before_decay = kMomentum ? __shfl_up(d, G, kWave) : 1.0;
    if (lane < (uint32_t)G) {
        before = D2{-0.0, -0.0};
        before_decay = 1.0;
    }
    return before;
}

// behind a barrier after heavy_sums: takes `state` from the round's start to its end, returns it as the lane's group finds it
template <int MODE, int WAVES, int G>
__device__ __forceinline__ D2 heavy_fold(D2 &state, const ExchangeOf<WAVES, G> &ex, uint32_t w, const D2 &before, double before_decay)
{
    constexpr bool kMomentum = MODE == kMomentumSeq;
    const uint32_t col_lane = lane_id() % G;
    D2 mine = state;
#pragma unroll
    for (int v = 0; v < WAVES; ++v) {
        if ((uint32_t)v == w) mine = state;
        const double fx = ex.sum[v][col_lane][0], fy = ex.sum[v][col_lane][1];
        const double dv = kMomentum ? ex.dec[v] : 1.0;
        state.x = kMomentum ? fma(dv, state.x, fx) : state.x + fx;
        state.y = kMomentum ? fma(dv, state.y, fy) : state.y + fy;
    }
    mine.x = kMomentum ? fma(before_decay, mine.x, before.x) : mine.x + before.x;
    mine.y = kMomentum ? fma(before_decay, mine.y, before.y) : mine.y + before.y;
    return mine;
}

// sum of the groups' steps over the workgroup, for every lane; one barrier, after ex was written
template <int WAVES, int G>
__device__ __forceinline__ D2 heavy_total(D2 acc, ExchangeOf<WAVES, G> &ex, uint32_t w)
{
    const uint32_t lane = lane_id(), col_lane = lane % G;
#pragma unroll
    for (int by = G; by < kWave; by <<= 1) {
        acc.x += __shfl_xor(acc.x, by, kWave);
        acc.y += __shfl_xor(acc.y, by, kWave);
    }
    if (lane < (uint32_t)G) {
        ex.sum[w][col_lane][0] = acc.x;
        ex.sum[w][col_lane][1] = acc.y;
    }
    __syncthreads();
    acc = D2{0, 0};
#pragma unroll
    for (int v = 0; v < WAVES; ++v) {
        acc.x += ex.sum[v][col_lane][0];
        acc.y += ex.sum[v][col_lane][1];
    }
    return acc;
}

}  // namespace ecrm
