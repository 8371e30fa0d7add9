// Reads of entries: plain gathers, reads while a server is down (its entries are decoded on the way, Sec. 3.2), and reads
// during a recovery (Sec. 3.4 "Training during recovery").
//
// During a recovery the paper serves a locked entry that has been updated meanwhile out of the buffer.  The buffer here
// holds updates, not entries, so the read applies them: the value returned is the stored entry with its waiting updates
// applied in arrival order -- what the entry will be once they have been replayed -- and an entry the failed server held
// that is not rebuilt yet is first decoded from its stripe (parity minus the other members, by increasing member, rounded
// to fp32 as the decoder stores it).  The waiting updates come grouped by entry.  An entry with waiting updates is
// answered once, for the first request that claims it, and copied to the others: every request for a hot entry walking its
// run by itself was what these reads took (65 536 half-Zipf requests among up to 60 000 waiting updates: 330 us on average,
// 157 to 900 from read to read).
//
// A gather is a flat copy: a lane moves 16 bytes of whatever row they belong to, so that rows of any width use all lanes,
// and a wave keeps several requests of both tables in flight.  (With one request of a wave at a time -- its key, then its
// row, then its accumulator, each a trip to memory -- 2^18 Zipf requests of 128 floats took 153 us; now 100, 444 MB that
// they cannot do without.  2^21 requests: 1135 and 688; 64 floats: 122 and 48; ten members to a stripe: 205 and 114.)
#include "long_runs.h"

namespace ecrm {

constexpr uint32_t kReadRun = 128;       // waiting updates from which on an entry is left to read_long_kernel
constexpr int kReadThreads = 256;
constexpr int kReadWaves = kReadThreads / kWave;

struct ReadArgs {
    const float *E, *A, *PE, *PA;
    const uint64_t *keys;
    uint64_t n;
    uint32_t per;            // consecutive requests of a wave, at most 64
    float *out_E, *out_A;    // out_A may be null
    Header *hdr;
    Geometry geo;
    Divider d4;              // by D / 4
    uint32_t lost;           // server whose entries are decoded, or none ...
    RecoveryView rv;         // ... unless their chunk is rebuilt already (in a recovery)
    // a recovery's waiting updates, sorted by entry: entry, gradient row in the pool
    const uint32_t *bk, *bi;
    const uint32_t *m_dev;   // how many there are (device word)
    const float *pool;
    uint32_t *leader;        // [m] at the head of a run: the request that answers for its entry
    uint32_t *place;         // [n] head of the run that a request's entry has, or kNoKey; null: there is no room for as many
    uint32_t *longs;         // head and leader of the runs that are left to read_long_kernel
};

// is the entry one that has to be decoded?
__device__ __forceinline__ bool is_lost(const ReadArgs &a, uint32_t g, uint32_t j)
{
    if (a.lost == ECRM_NO_SERVER || a.geo.dS.mod(g + 1u + j) != a.lost) return false;
    return !a.rv.active || a.rv.dspc.div(g) >= a.rv.next;
}

__device__ __forceinline__ void store4(float *p, float4 v)               // written once, read by somebody else later
{
    typedef float f4 __attribute__((ext_vector_type(4)));
    __builtin_nontemporal_store(__builtin_bit_cast(f4, v), (f4 *)p);
}

// The requests of a wave that are handled alike: lane's request (row x, the i-th of the wave) if `mine`.
__device__ __forceinline__ uint32_t collect(bool mine, uint32_t x, uint32_t i, uint2 *list)
{
    const unsigned long long m = __ballot(mine);
    if (mine) list[__popcll(m & bits_below(lane_id()))] = uint2{x, i};
    __builtin_amdgcn_wave_barrier();
    return (uint32_t)__popcll(m);
}

// rows list[..].x of the source tables to rows first + list[..].y of the outputs
__device__ __forceinline__ void copy_rows(const ReadArgs &a, const float *from_E, const float *from_A, uint64_t first,
                                          const uint2 *list, uint32_t cnt)
{
    constexpr uint32_t U = 4;                            // (2, 4, 8: 101, 102, 103 us)
    const uint32_t lane = lane_id(), D = a.geo.D, total = cnt * (D / 4u);
    for (uint32_t u0 = 0; u0 < total; u0 += U * kWave) {
        float4 e[U], s[U];
        size_t to[U];
#pragma unroll
        for (uint32_t q = 0; q < U; ++q) {
            const uint32_t u = min(u0 + q * kWave + lane, total - 1u), r = a.d4.div(u), c = (u - r * a.d4.d) * 4u;
            const uint2 what = list[r];
            const size_t from = (size_t)what.x * D + c;
            to[q] = (first + what.y) * D + c;
            e[q] = load4(from_E + from);
            if (a.out_A) s[q] = load4(from_A + from);
        }
#pragma unroll
        for (uint32_t q = 0; q < U; ++q) {
            if (u0 + q * kWave + lane >= total) continue;
            store4(a.out_E + to[q], e[q]);
            if (a.out_A) store4(a.out_A + to[q], s[q]);
        }
    }
}

__device__ __forceinline__ void subtract4(double (&v)[4], float4 o)
{
    v[0] -= (double)o.x;
    v[1] -= (double)o.y;
    v[2] -= (double)o.z;
    v[3] -= (double)o.w;
}
// lost entries: their parity minus the other members, by increasing member
template <bool BOTH>
__device__ __forceinline__ void decode_rows(const ReadArgs &a, uint64_t first, const uint2 *list, uint32_t cnt)
{
    constexpr uint32_t U = 4;                            // members in flight
    const uint32_t lane = lane_id(), D = a.geo.D, k = a.geo.k, total = cnt * (D / 4u);
    for (uint32_t u = lane; u < total; u += kWave) {
        const uint32_t r = a.d4.div(u), c = (u - r * a.d4.d) * 4u;
        const uint2 what = list[r];
        const uint32_t g = a.geo.dk.div(what.x), j = what.x - g * k;
        const float4 p[2] = {load4(a.PE + (size_t)g * D + c), BOTH ? load4(a.PA + (size_t)g * D + c) : float4{0, 0, 0, 0}};
        double v[2][4];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            v[t][0] = (double)p[t].x;
            v[t][1] = (double)p[t].y;
            v[t][2] = (double)p[t].z;
            v[t][3] = (double)p[t].w;
        }
        for (uint32_t m0 = 0; m0 < k - 1u; m0 += U) {    // the survivors: member m, or m + 1 from the lost one on
            float4 o[2][U];
#pragma unroll
            for (uint32_t q = 0; q < U; ++q) {
                const uint32_t m = min(m0 + q, k - 2u);
                const size_t from = ((size_t)g * k + (m < j ? m : m + 1u)) * D + c;
                o[0][q] = load4(a.E + from);
                if (BOTH) o[1][q] = load4(a.A + from);
            }
#pragma unroll
            for (uint32_t q = 0; q < U; ++q) {
                if (m0 + q >= k - 1u) continue;
                subtract4(v[0], o[0][q]);
                if (BOTH) subtract4(v[1], o[1][q]);
            }
        }
        const size_t to = (first + what.y) * D + c;
        store4(a.out_E + to, float4{(float)v[0][0], (float)v[0][1], (float)v[0][2], (float)v[0][3]});
        if (BOTH) store4(a.out_A + to, float4{(float)v[1][0], (float)v[1][1], (float)v[1][2], (float)v[1][3]});
    }
}

// first position of the sorted keys [0, m) that is not below x, a lane's own search: three probes a step
__device__ __forceinline__ uint32_t first_not_below(const uint32_t *bk, uint32_t m, uint32_t x)
{
    uint32_t lo = 0, end = m;                            // the answer lies in [lo, end]
    while (lo < end) {
        const uint32_t step = (end - lo + 3u) / 4u;
        uint32_t below = 0;
#pragma unroll
        for (uint32_t q = 1; q <= 3; ++q) {
            const uint32_t p = lo + q * step - 1u;
            below += bk[min(p, m - 1u)] < x && p < end ? 1u : 0u;
        }
        lo += below * step;
        if (below < 3u) end = min(end, lo + step - 1u);
    }
    return lo;
}

// head of the run of x, an entry of the tables, among m waiting updates
__device__ __forceinline__ uint32_t waiting_run(const ReadArgs &a, uint32_t m, uint32_t x)
{
    if (!m || !held_back(a.rv, x, a.geo.dk, a.geo.dS)) return kNoKey;
    const uint32_t p = first_not_below(a.bk, m, x);
    return p < m && a.bk[p] == x ? p : kNoKey;
}

// One entry with fewer than kReadRun waiting updates, by a wave, for request i (all wave-uniform).
template <int MODE>
__device__ __forceinline__ void read_run(const ReadArgs &a, uint32_t m, uint32_t pos, uint32_t x, uint64_t i)
{
    const uint32_t D = a.geo.D, k = a.geo.k, lane = lane_id(), g = a.geo.dk.div(x), j = x - g * k;
    const RuleParams rp = rule_params(a.geo);
    const bool decode = is_lost(a, g, j);
    for (uint32_t col0 = 0; col0 < D; col0 += 128u) {
        D2 e, s0;
        if (decode) {
            e = widen2(ld2<0>(row_f32(a.PE, g, D, col0), 0));
            s0 = widen2(ld2<0>(row_f32(a.PA, g, D, col0), 0));
            for (uint32_t m0 = 0; m0 < k - 1u; m0 += 4u) {
                float2 oe[4], os[4];
#pragma unroll
                for (uint32_t u = 0; u < 4u; ++u) {
                    const uint32_t mth = min(m0 + u, k - 2u), row = g * k + (mth < j ? mth : mth + 1u);
                    oe[u] = ld2<0>(row_f32(a.E, row, D, col0), 0);
                    os[u] = ld2<0>(row_f32(a.A, row, D, col0), 0);
                }
#pragma unroll
                for (uint32_t u = 0; u < 4u; ++u) {
                    if (m0 + u >= k - 1u) continue;
                    e.x -= (double)oe[u].x; e.y -= (double)oe[u].y;
                    s0.x -= (double)os[u].x; s0.y -= (double)os[u].y;
                }
            }
            e = widen2(narrow2(e));
            s0 = widen2(narrow2(s0));
        } else {
            e = widen2(ld2<0>(row_f32(a.E, x, D, col0), 0));
            s0 = widen2(ld2<0>(row_f32(a.A, x, D, col0), 0));
        }
        D2 G = s0, acc = D2{0, 0};
        for (uint32_t p = pos; p < m; p += kWave) {      // 64 places at a time, U gradients in flight
            constexpr uint32_t U = 16;
            const bool in = p + lane < m;
            const uint32_t wk = in ? a.bk[p + lane] : kNoKey, wi = in ? a.bi[p + lane] : 0u;
            const unsigned long long other = ~__ballot(wk == x);
            const uint32_t cnt = other ? lowest_bit(other) : (uint32_t)kWave;     // leading run of x
            for (uint32_t u0 = 0; u0 < cnt; u0 += U) {
                float2 gr[U];
#pragma unroll
                for (uint32_t u = 0; u < U; ++u)
                    gr[u] = ld2<0>(row_f32(a.pool, from_lane(wi, min(u0 + u, cnt - 1u)), D, col0), 0);
#pragma unroll
                for (uint32_t u = 0; u < U; ++u)
                    if (u0 + u < cnt) item2<MODE>(G, acc, gr[u], rp);
            }
            if (cnt < (uint32_t)kWave) break;
        }
        const rsrc_t oe = __builtin_amdgcn_make_buffer_rsrc(a.out_E + (size_t)i * D + col0, 0, (int)((D - col0) * 4u), kRsrcFlags);
        st2(oe, 0, narrow2(D2{e.x - acc.x, e.y - acc.y}));
        if (a.out_A) {
            const rsrc_t oa = __builtin_amdgcn_make_buffer_rsrc(a.out_A + (size_t)i * D + col0, 0, (int)((D - col0) * 4u), kRsrcFlags);
            st2(oa, 0, narrow2(G));
        }
    }
}

// A wave's `per` requests: those of stored entries are copied, those of lost ones decoded, and of those with waiting
// updates (WAITING: there may be some) the first to claim an entry has it answered.
template <bool WAITING, int MODE>
__global__ __launch_bounds__(kReadThreads) void read_entries_kernel(ReadArgs a)
{
    __shared__ uint2 s_list[kReadWaves][kWave];
    const uint32_t lane = lane_id();
    uint2 *list = s_list[threadIdx.x / kWave];
    const uint64_t first = ((uint64_t)blockIdx.x * kReadWaves + uniform(threadIdx.x / kWave)) * a.per;
    if (first >= a.n) return;
    const uint32_t cnt = (uint32_t)(a.n - first < a.per ? a.n - first : a.per);
    const uint64_t key = lane < cnt ? a.keys[first + lane] : 0ull;
    const uint32_t x = (uint32_t)key;
    const bool bad = key >= (uint64_t)a.geo.rows, valid = lane < cnt && !bad;
    if (bad) atomicOr(&a.hdr->err_sticky, 1u);
    const uint32_t g = a.geo.dk.div(x), j = x - g * a.geo.k;
    uint32_t pos = kNoKey;                               // head of the entry's waiting run
    bool claimed = false;
    const uint32_t m = WAITING ? uniform(*a.m_dev) : 0u;
    if (WAITING) {
        if (valid) pos = waiting_run(a, m, x);
        if (pos != kNoKey) {
            claimed = atomicCAS(&a.leader[pos], kNoKey, (uint32_t)(first + lane)) == kNoKey;
            if (claimed && pos + kReadRun <= m && a.bk[pos + kReadRun - 1u] == x) {
                const uint32_t at = atomicAdd(&a.hdr->n_reads, 1u);
                a.longs[2u * at] = pos;                  // at most m / kReadRun of them
                a.longs[2u * at + 1u] = (uint32_t)(first + lane);
                claimed = false;
            }
        }
        if (lane < cnt && a.place) a.place[first + lane] = pos;
    }
    const bool lost = valid && pos == kNoKey && is_lost(a, g, j);
    const uint32_t plain = collect(valid && pos == kNoKey && !lost, x, lane, list);
    if (plain) copy_rows(a, a.E, a.A, first, list, plain);
    __builtin_amdgcn_wave_barrier();
    const uint32_t dec = collect(lost, x, lane, list);
    if (dec) {
        if (a.out_A) decode_rows<true>(a, first, list, dec);
        else decode_rows<false>(a, first, list, dec);
    }
    if (WAITING) {
        for (unsigned long long todo = __ballot(claimed); todo; todo &= todo - 1ull) {
            const uint32_t l = lowest_bit(todo);
            read_run<MODE>(a, m, from_lane(pos, l), from_lane(x, l), first + l);
        }
    }
}

// before the requests are looked at: no entry is claimed, no run is listed
__global__ __launch_bounds__(kReadThreads) void read_begin_kernel(Header *hdr, const uint32_t *m_dev, uint32_t *leader)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) hdr->n_reads = hdr->read_ticket = 0;
    const uint32_t m = *m_dev, i = (blockIdx.x * kReadThreads + threadIdx.x) * 4u;
    if (i < m) *(uint4 *)(leader + i) = uint4{kNoKey, kNoKey, kNoKey, kNoKey};      // room for a multiple of four
}

// The entries with many waiting updates: (entry, 16 columns) per workgroup.
template <int MODE>
__global__ __launch_bounds__(kHeavyThreads) void read_long_kernel(ReadArgs a)
{
    constexpr int T = kHeavyT;
    __shared__ HeavyExchange s_ex[2];
    __shared__ uint32_t s_job;
    const uint32_t D = a.geo.D, k = a.geo.k, lane = lane_id(), w = uniform(threadIdx.x / kWave);
    const uint32_t col_lane = lane & 7u, sub = w * 8u + lane / 8u, ncg = (D + kHeavyCols - 1) / kHeavyCols;
    const RuleParams rp = rule_params(a.geo);
    const uint32_t m = uniform(*a.m_dev), jobs = uniform(a.hdr->n_reads) * ncg;
    for (;;) {
        if (threadIdx.x == 0) s_job = jobs ? atomicAdd(&a.hdr->read_ticket, 1u) : 0u;
        __syncthreads();
        const uint32_t job = uniform(s_job);
        if (job >= jobs) break;                          // every workgroup draws one number past the last job
        const uint32_t p = uniform(a.longs[2u * (job / ncg)]), i = uniform(a.longs[2u * (job / ncg) + 1u]);
        const uint32_t col = job % ncg * kHeavyCols + 2u * col_lane;
        const bool live = col < D;                       // D is a multiple of 4: both columns or none
        const uint32_t x = uniform(a.bk[p]), g = a.geo.dk.div(x), j = x - g * k;
        uint32_t lo = p, hi = m;                         // bk[lo] is x; hi: the first that is not
        while (hi - lo > 1u) {
            const uint32_t step = (hi - lo + kWave - 1) / kWave, probe = lo + (lane + 1u) * step;
            const uint32_t in = (uint32_t)__popcll(__ballot(probe < hi && a.bk[min(probe, m - 1u)] == x));
            const uint32_t out = lo + (in + 1u) * step;
            lo += in * step;
            if (in < (uint32_t)kWave && out < hi) hi = out;
        }
        const uint32_t L = hi - p;
        const uint32_t *run = a.bi + p;
        float2 gr[T], nx[T];
        uint32_t i0, i1;
        heavy_indices(run, L, sub * T + 2u * col_lane, i0, i1);
        heavy_rows<T>(nx, a.pool, D, col, live, i0, i1, lane, sub * T, L);
        heavy_indices(run, L, 64u * T + sub * T + 2u * col_lane, i0, i1);
        D2 e = D2{0, 0}, s0 = D2{0, 0};
        if (live) {
            if (is_lost(a, g, j)) {
                e = widen2(*(const float2 *)(a.PE + (size_t)g * D + col));
                s0 = widen2(*(const float2 *)(a.PA + (size_t)g * D + col));
#pragma unroll 4
                for (uint32_t mth = 0; mth < k - 1u; ++mth) {
                    const size_t row = ((size_t)g * k + (mth < j ? mth : mth + 1u)) * D + col;
                    const float2 oe = *(const float2 *)(a.E + row), os = *(const float2 *)(a.A + row);
                    e.x -= (double)oe.x; e.y -= (double)oe.y;
                    s0.x -= (double)os.x; s0.y -= (double)os.y;
                }
                e = widen2(narrow2(e));
                s0 = widen2(narrow2(s0));
            } else {
                e = widen2(*(const float2 *)(a.E + (size_t)x * D + col));
                s0 = widen2(*(const float2 *)(a.A + (size_t)x * D + col));
            }
        }
        D2 state = s0, acc = D2{0, 0};
        uint32_t buf = 0;                                // half of s_ex: changes with every exchange
        for (uint32_t r0 = 0; r0 < L; r0 += 64u * T) {
            const uint32_t off = r0 + sub * T, cnt = off < L ? min((uint32_t)T, L - off) : 0u;
#pragma unroll
            for (int u = 0; u < T; ++u) gr[u] = nx[u];
            if (r0 + 64u * T < L) {
                heavy_rows<T>(nx, a.pool, D, col, live, i0, i1, lane, off + 64u * T, L);
                heavy_indices(run, L, off + 128u * T + 2u * col_lane, i0, i1);
            }
            double ed;
            const D2 ex = heavy_sums<MODE>(gr, cnt, rp, s_ex[buf], w, ed);
            __syncthreads();
            D2 mine = heavy_fold<MODE>(state, s_ex[buf], w, ex, ed);
#pragma unroll
            for (int u = 0; u < T; ++u) {
                if ((uint32_t)u < cnt) item2<MODE>(mine, acc, gr[u], rp);
            }
            buf ^= 1u;
        }
        acc = heavy_total(acc, s_ex[buf], w);
        if (live && sub == 0) {
            *(float2 *)(a.out_E + (size_t)i * D + col) = narrow2(D2{e.x - acc.x, e.y - acc.y});
            if (a.out_A) *(float2 *)(a.out_A + (size_t)i * D + col) = narrow2(state);
        }
        __syncthreads();                                 // s_ex and s_job are free for the next job
    }
}

// The requests whose entries were answered for another one.  Where there was no room for the places of their runs they are
// looked up once more: 2^18 requests of a context made for batches of 2048 138 us; when such a read was cut into parts of 2048,
// of four launches each, 2367.
__global__ __launch_bounds__(kReadThreads) void read_shared_kernel(ReadArgs a)
{
    __shared__ uint2 s_list[kReadWaves][kWave];
    const uint32_t lane = lane_id();
    uint2 *list = s_list[threadIdx.x / kWave];
    const uint64_t first = ((uint64_t)blockIdx.x * kReadWaves + uniform(threadIdx.x / kWave)) * a.per;
    if (first >= a.n) return;
    uint32_t from = kNoKey;
    if (lane < a.per && first + lane < a.n) {
        uint32_t pos = kNoKey;
        if (a.place) {
            pos = a.place[first + lane];
        } else {
            const uint64_t key = a.keys[first + lane];
            if (key < (uint64_t)a.geo.rows) pos = waiting_run(a, *a.m_dev, (uint32_t)key);
        }
        if (pos != kNoKey) from = a.leader[pos];
    }
    const uint32_t cnt = collect(from != kNoKey && from != (uint32_t)(first + lane), from, lane, list);
    if (cnt) copy_rows(a, a.out_E, a.out_A, first, list, cnt);
}

// ================================================================================================
// host side
// ================================================================================================

// Consecutive requests of a wave: as many as make the launch thirty-two waves to a compute unit
// (2^18 requests: 100.4 us, 102.0 with sixteen, 102.1 with eight).
static uint32_t requests_per_wave(uint64_t n, int cus)
{
    const uint64_t want = n / ((uint64_t)cus * 32u);
    return want < 4u ? 4u : want > (uint64_t)kWave ? (uint32_t)kWave : (uint32_t)want;
}

static ReadArgs read_args(const Scratch &s, const Geometry &g, const float *E, const float *A, const float *PE, const float *PA,
                          uint32_t lost)
{
    ReadArgs a = {};
    a.E = E; a.A = A; a.PE = PE; a.PA = PA;
    a.hdr = s.hdr; a.geo = g; a.d4 = make_divider(g.D / 4u); a.lost = lost;
    return a;
}

// Requests that are answered by one set of launches: as many threads, which is what a launch can have.
constexpr uint64_t kReadSlice = 1u << 30;

static dim3 read_grid(const ReadArgs &a)
{
    const uint64_t waves = (a.n + a.per - 1) / a.per;
    return dim3((uint32_t)((waves + kReadWaves - 1) / kReadWaves));
}

// the requests from the at-th of n on
static void next_slice(ReadArgs &a, uint64_t at, uint64_t n, const uint64_t *keys, float *out_E, float *out_A, int cus)
{
    a.keys = keys + at;
    a.n = n - at < kReadSlice ? n - at : kReadSlice;
    a.out_E = out_E + at * a.geo.D;
    a.out_A = out_A ? out_A + at * a.geo.D : nullptr;
    a.per = requests_per_wave(a.n, cus);
}

void launch_degraded_read(const Scratch &s, const Geometry &g, const float *E, const float *A, const float *PE,
                          const float *PA, const uint64_t *keys, uint64_t n, uint32_t lost, float *out_E,
                          float *out_A, int cus, hipStream_t st)
{
    ReadArgs a = read_args(s, g, E, A, PE, PA, lost);
    for (uint64_t at = 0; at < n; at += kReadSlice) {
        next_slice(a, at, n, keys, out_E, out_A, cus);
        hipLaunchKernelGGL((read_entries_kernel<false, kAdagradSeq>), read_grid(a), dim3(kReadThreads), 0, st, a);
    }
}

template <int MODE>
static void recovery_read_slice(const ReadArgs &a, uint32_t cap, bool cleared, int cus, hipStream_t st)
{
    if (!cleared)
        hipLaunchKernelGGL(read_begin_kernel, dim3((cap + 4u * kReadThreads - 1) / (4u * kReadThreads)), dim3(kReadThreads), 0, st,
                           a.hdr, a.m_dev, a.leader);
    hipLaunchKernelGGL((read_entries_kernel<true, MODE>), read_grid(a), dim3(kReadThreads), 0, st, a);
    const uint32_t jobs = cap / kReadRun * ((a.geo.D + kHeavyCols - 1) / kHeavyCols);         // at most
    if (jobs) hipLaunchKernelGGL(read_long_kernel<MODE>, dim3(min(jobs, (uint32_t)cus)), dim3(kHeavyThreads), 0, st, a);
    hipLaunchKernelGGL(read_shared_kernel, read_grid(a), dim3(kReadThreads), 0, st, a);
}

// bk, bi: the waiting updates, as launch_sort left them (of a buffer of `cap` of them); leader: room for as many, and if it and
// the header's fields are cleared already; max_batch: what the scratch buffer serves
void launch_recovery_read(const Scratch &s, const Geometry &g, const RecoveryView &rv, const float *E, const float *A,
                          const float *PE, const float *PA, const uint64_t *keys, uint64_t n, const uint32_t *bk,
                          const uint32_t *bi, uint32_t *leader, bool cleared, const uint32_t *m_dev, uint32_t cap,
                          const float *pool, uint32_t max_batch, float *out_E, float *out_A, int cus, hipStream_t st)
{
    ReadArgs a = read_args(s, g, E, A, PE, PA, rv.server);
    a.rv = rv; a.bk = bk; a.bi = bi; a.m_dev = m_dev; a.pool = pool;
    a.place = n <= max_batch ? s.keys[bk == s.keys[0] ? 1 : 0] : nullptr;   // the sort is done with the other halves of its buffers
    a.leader = leader;
    a.longs = s.active;
    for (uint64_t at = 0; at < n; at += kReadSlice) {
        next_slice(a, at, n, keys, out_E, out_A, cus);
        if (at) cleared = false;                             // the leaders of the requests before
        if (g.mode == kMomentumSeq) recovery_read_slice<kMomentumSeq>(a, cap, cleared, cus, st);
        else recovery_read_slice<kAdagradSeq>(a, cap, cleared, cus, st);       // a recovery takes no combined rule
    }
}

}  // namespace ecrm
