// The smallest batches (up to kDirectBatch updates) in one launch.  What bounds them is the number of dependent steps and
// nothing else: through the three launches of buckets.hip 2048 uniform updates, 9 MB, took 16.2 us, now 10.4.  Here every workgroup
// reads all keys of the batch -- up to 24 KB that come out of the L2 --, picks its bucket's and goes on as bucket_apply does with a list
// in LDS.  Since all workgroups see all keys, they agree on what is long without a word: a stripe of kDirectLong updates may be left
// to workgroups that look at the long buckets only, eight columns of such a stripe at a time (direct_by_columns).  One more workgroup
// does what concerns the batch as a whole: the load counts and the header.  Nothing of the scratch buffer but the header is used.
#include "lists.h"

namespace ecrm {

constexpr int kDirectLanes = 4;                                        // that hold two columns each of an update of a long stripe
// Keys of a thread, K below: a variant with fewer for the smaller ones of these batches (2048 uniform updates 9.9 us, with the
// larger one 10.9; branches around the loads that a batch does not need cost more than the loads: 12.1).
constexpr uint32_t kDirectKeys = kDirectBatch / kBucketThreads, kDirectFewKeys = 8;
static_assert(kDirectKeys * kBucketWaves <= (uint32_t)kWave, "a lane to a wave's share of 64 keys");

struct DirectArgs : RowArgs {
    const uint64_t *keys;
    Header *hdr;
    u64 *load_data, *load_parity;
    uint32_t *rejected;
    uint32_t n, buckets, clear_sticky;
    uint32_t stripes, sure;      // of the table; direct_sure
};

template <uint32_t K>
struct DirectShared {
    static constexpr uint32_t kItems = K * kBucketThreads, kLongs = kItems / kDirectLong;
    __align__(16) u64 item[kItems];
    union {
        __align__(16) u64 tmp[kItems];
        ExchangeOf<kBucketWaves, kDirectLanes> ex[2];
    };
    union {
        FewRows few;                                                    // before the list is walked
        ListShared<kItems> list;
    };
    uint32_t in_bucket[kItems / 8u];                              // items of each bucket
    uint32_t found[kLongs], longs[kLongs], n_found, count[K * kBucketWaves];
    uint32_t n_long, n_long_items, n_empty;
};

// the thread's keys of the batch: positions threadIdx.x, + kBucketThreads, ...
template <uint32_t K>
struct Keys {
    uint32_t row[K];
    bool bad;
};
template <uint32_t K>
__device__ __forceinline__ Keys<K> read_keys(const DirectArgs &a)
{
    Keys<K> k;
    u64 key[K];
#pragma unroll
    for (uint32_t r = 0; r < K; ++r) {
        const uint32_t i = r * kBucketThreads + threadIdx.x;
        key[r] = i < a.n ? a.keys[i] : 0ull;
    }
    k.bad = false;
#pragma unroll
    for (uint32_t r = 0; r < K; ++r) {
        k.row[r] = (uint32_t)key[r];
        k.bad |= key[r] >= (u64)a.geo.rows;
    }
    return k;
}

// the items of bucket b, sorted; returns how many they are
template <uint32_t K>
__device__ __forceinline__ uint32_t collect(const DirectArgs &a, const Keys<K> &k, DirectShared<K> &sh, uint32_t b)
{
    const uint32_t lane = lane_id(), w = uniform(threadIdx.x / kWave);
    u64 mine[K];                                              // in arrival order: key by key, wave by wave
#pragma unroll
    for (uint32_t r = 0; r < K; ++r) {
        const uint32_t i = r * kBucketThreads + threadIdx.x;
        mine[r] = __ballot(i < a.n && bucket_of(a.geo.dk.div(k.row[r]), a.buckets) == b);
        if (lane == 0) sh.count[r * kBucketWaves + w] = (uint32_t)__popcll(mine[r]);
    }
    __syncthreads();
    uint32_t incl = lane < K * kBucketWaves ? sh.count[lane] : 0u;
    const uint32_t own = incl;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t up = __shfl_up(incl, d, kWave);
        if (lane >= (uint32_t)d) incl += up;
    }
    const uint32_t m = from_lane(incl, kWave - 1u), before = incl - own;
#pragma unroll
    for (uint32_t r = 0; r < K; ++r) {
        const uint32_t at = from_lane(before, r * kBucketWaves + w) + (uint32_t)__popcll(mine[r] & bits_below(lane));
        if ((mine[r] >> lane) & 1ull) sh.item[at] = ((u64)k.row[r] << 32) | (r * kBucketThreads + threadIdx.x);
    }
    __syncthreads();
    // counted from 129 items on in the larger variant: 3000 Zipf on 2^16 rows 21.1 us, so from 257 on 21.4; 900 15.6, 15.3
    if (m) sort_items(sh.item, sh.tmp, m, true, sh.few, K > kDirectFewKeys ? kFewLeast / 2u : kFewLeast);
    return m;
}

// The buckets of `least` items or more (at least kDirectLong), their numbers, ascending, in sh.longs; and those that have none.
struct Buckets { uint32_t found, empty; };
template <uint32_t K>
__device__ __forceinline__ Buckets find_long(const DirectArgs &a, const Keys<K> &k, DirectShared<K> &sh, uint32_t least)
{
    for (uint32_t b = threadIdx.x; b < a.buckets; b += kBucketThreads) sh.in_bucket[b] = 0;
    if (threadIdx.x == 0) sh.n_found = sh.n_empty = 0;
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < K; ++r) {
        const uint32_t i = r * kBucketThreads + threadIdx.x;
        if (i < a.n) atomicAdd(&sh.in_bucket[bucket_of(a.geo.dk.div(k.row[r]), a.buckets)], 1u);
    }
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < a.buckets; b += kBucketThreads) {
        const uint32_t m = sh.in_bucket[b];
        const u64 none = __ballot(m == 0);
        if (lane_id() == 0 && none) atomicAdd(&sh.n_empty, (uint32_t)__popcll(none));
        if (m >= least) sh.found[atomicAdd(&sh.n_found, 1u)] = b;
    }
    __syncthreads();
    const uint32_t nb = uniform(sh.n_found);
    if (threadIdx.x < nb) {
        uint32_t rank = 0;
        for (uint32_t i = 0; i < nb; ++i) rank += sh.found[i] < sh.found[threadIdx.x] ? 1u : 0u;
        sh.longs[rank] = sh.found[threadIdx.x];
    }
    __syncthreads();
    return Buckets{nb, uniform(sh.n_empty)};
}

// Whether the long stripes of a bucket, whose list of m items this is, are left to the workgroups that take them by columns: the
// same for all that look at it.  By a whole workgroup.
template <int MODE, uint32_t K>
__device__ __forceinline__ bool by_columns(const DirectArgs &a, DirectShared<K> &sh, uint32_t m)
{
    if (m >= a.sure) return true;
    const uint32_t x = item_row(sh.item[m / 2u]);                       // a row that has nearly all of them
    if (x == item_row(sh.item[m / 8u]) || x == item_row(sh.item[m - 1u - m / 8u])) return true;
    return direct_by_columns(count_runs(sh.item, m, sh.count), a.n, a.stripes, a.geo.D, Rule<MODE>::combine);
}

// What concerns the batch as a whole: one workgroup.
template <int MODE, uint32_t K>
__device__ __forceinline__ void direct_batch(const DirectArgs &a, const Keys<K> &k, bool bad, DirectShared<K> &sh)
{
    const uint32_t tid = threadIdx.x, S = a.geo.S;
    if (tid == 0) {
        begin_batch(a.hdr, a.n, a.clear_sticky != 0);
        a.hdr->n_hot = 0;
        if (bad) {
            a.hdr->batch_bad = 1;
            a.hdr->err_sticky |= 1u;
        }
        if (a.rejected) *a.rejected = bad ? 1u : 0u;
    }
    if (bad) return;
    if (!Rule<MODE>::combine) {
        for (uint32_t i = tid; i < 2 * S; i += kBucketThreads) sh.list.srv[i] = 0;
        __syncthreads();
#pragma unroll
        for (uint32_t r = 0; r < K; ++r) {
            const uint32_t i = r * kBucketThreads + tid;
            if (i >= a.n) continue;
            const uint32_t g = a.geo.dk.div(k.row[r]), j = k.row[r] - g * a.geo.k;
            atomicAdd(&sh.list.srv[a.geo.dS.mod(g + 1 + j)], 1u);
            atomicAdd(&sh.list.srv[S + a.geo.dS.mod(g)], 1u);
        }
        __syncthreads();
        for (uint32_t i = tid; i < 2 * S; i += kBucketThreads) {
            u64 *to = i < S ? a.load_data : a.load_parity;
            if (to) to[i < S ? i : i - S] += sh.list.srv[i];
        }
    }
    if (a.n <= kLongRun) return;
    if (tid == 0) sh.n_long = sh.n_long_items = 0;                      // rows that ecrm_batch_stats reports
    const uint32_t nb = find_long(a, k, sh, kLongRun + 1u).found;
    for (uint32_t i = 0; i < nb; ++i) {
        const uint32_t m = collect(a, k, sh, uniform(sh.longs[i]));
        for (uint32_t p = tid; p + kLongRun < m; p += kBucketThreads) {
            const uint32_t x = item_row(sh.item[p]);
            if ((p && item_row(sh.item[p - 1]) == x) || item_row(sh.item[p + kLongRun]) != x) continue;
            uint32_t last = p + kLongRun, out = m;                      // of the run, and behind it
            while (out - last > 1u) {
                const uint32_t mid = (last + out) / 2u;
                if (item_row(sh.item[mid]) == x) last = mid; else out = mid;
            }
            atomicAdd(&sh.n_long, 1u);
            atomicAdd(&sh.n_long_items, out - p);
        }
        __syncthreads();
    }
    if (tid == 0) {
        a.hdr->n_long = sh.n_long;
        a.hdr->n_long_items = sh.n_long_items;
    }
}

// The long stripes, eight columns at a time: a workgroup takes consecutive jobs -- a bucket, eight columns --, mostly of one
// bucket, whose list it makes once.  own: of a workgroup whose bucket is empty the bucket, otherwise kNoKey.
template <int MODE, bool PARITY, uint32_t K>
__device__ __forceinline__ void direct_columns(const DirectArgs &a, const Keys<K> &k, DirectShared<K> &sh, uint32_t own)
{
    const Divider dk = a.geo.dk;
    const Buckets longs = find_long(a, k, sh, kDirectLong);
    const uint32_t groups = direct_groups(a.geo.D), jobs = longs.found * groups, workers = direct_workers(jobs, longs.empty);
    const uint32_t turns = (jobs + workers - 1u) / workers;
    uint32_t worker = blockIdx.x - 1u;
    if (own != kNoKey) {                                                // these come behind the others, in their order
        worker = kDirectWorkers;
        for (uint32_t b = lane_id(); b - lane_id() < own; b += kWave)
            worker += (uint32_t)__popcll(__ballot(b < own && sh.in_bucket[b] == 0));
    }
    uint32_t have = kNoKey, m = 0;
    const uint32_t end_job = min((worker + 1u) * turns, jobs);
    bool mine = false;
    for (uint32_t job = worker * turns; job < end_job; ++job) {
        const uint32_t b = uniform(sh.longs[job / groups]);
        if (b != have) {
            m = collect(a, k, sh, b);
            have = b;
            mine = by_columns<MODE>(a, sh, m);
        }
        for (uint32_t p = 0; mine && p + kDirectLong <= m;) {
            const uint32_t g = dk.div(uniform(item_row(sh.item[p])));
            uint32_t end = p;
            for (;;) {
                const uint32_t q = end + lane_id();
                const u64 other = __ballot(q >= m || dk.div(item_row(sh.item[min(q, m - 1u)])) != g);
                if (other) {
                    end += lowest_bit(other);
                    break;
                }
                end += kWave;
            }
            if (end - p >= kDirectLong) stripe_columns<MODE, PARITY>(a, sh.item, p, end, job % groups, sh.ex);
            p = end;
        }
    }
}

static_assert(kDirectLong > (uint32_t)kWave, "such a stripe ends in no window");

// Two workgroups of a compute unit are all there are: more would only spill (2048 Zipf on 1024 rows 15.6 us, with room for four 17.9).
template <int NC, int MODE, bool PARITY, uint32_t K>
__global__ __launch_bounds__(kBucketThreads, 2) void direct_kernel(DirectArgs a)
{
    __shared__ DirectShared<K> sh;
    const Keys<K> k = read_keys<K>(a);
    const bool bad = __syncthreads_or(k.bad);
    if (blockIdx.x == 0) {
        direct_batch<MODE>(a, k, bad, sh);
        return;
    }
    if (bad) return;
    const uint32_t b = blockIdx.x > kDirectWorkers ? blockIdx.x - 1u - kDirectWorkers : kNoKey;
    if (b != kNoKey) {
        const uint32_t m = collect(a, k, sh, b);
        if (m) {
            if (Rule<MODE>::combine) count_list(a.geo, sh.item, m, sh.list.srv, a.load_data, a.load_parity);
            uint32_t least = ~0u;
            if (__builtin_expect(m >= kDirectLong, 0) && by_columns<MODE>(a, sh, m)) {
                if (a.geo.dk.div(item_row(sh.item[0])) == a.geo.dk.div(item_row(sh.item[m - 1u]))) return;      // nothing else
                least = kDirectLong;
            }
            apply_list<NC, MODE, PARITY, false, false>(a, sh.item, m, 0u, least, sh.list, (double *)sh.tmp);
            return;
        }
        // an empty bucket's workgroup helps where there may be more jobs than the others take at once
        if (min(a.n / kDirectLong, a.stripes) * direct_groups(a.geo.D) <= kDirectWorkers) return;
    }
    direct_columns<MODE, PARITY>(a, k, sh, b);
}

// ================================================================================================
// host side
// ================================================================================================

template <int NC, int MODE>
static void direct_for(const DirectArgs &a, bool parity, hipStream_t st)
{
    const dim3 grid(1u + kDirectWorkers + a.buckets), block(kBucketThreads);
    if (a.n <= kDirectFewKeys * kBucketThreads) {
        if (parity) hipLaunchKernelGGL((direct_kernel<NC, MODE, true, kDirectFewKeys>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((direct_kernel<NC, MODE, false, kDirectFewKeys>), grid, block, 0, st, a);
    } else {
        if (parity) hipLaunchKernelGGL((direct_kernel<NC, MODE, true, kDirectKeys>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((direct_kernel<NC, MODE, false, kDirectKeys>), grid, block, 0, st, a);
    }
}

void launch_direct(Header *hdr, const Geometry &g, float *E, float *A, float *PE, float *PA, unsigned long long *load_data,
                   unsigned long long *load_parity, const uint64_t *keys, uint32_t *rejected, const float *grads, uint32_t n,
                   bool clear_sticky, hipStream_t st)
{
    DirectArgs a;
    a.E = E; a.A = A; a.PE = PE; a.PA = PA; a.grads = grads; a.geo = g;
    a.keys = keys; a.hdr = hdr; a.load_data = load_data; a.load_parity = load_parity; a.rejected = rejected;
    a.n = n; a.buckets = direct_buckets(n); a.clear_sticky = clear_sticky ? 1u : 0u;
    a.stripes = g.dk.div(g.rows);
    a.sure = direct_sure(n, a.stripes, g.k, g.D, (g.mode & 2u) != 0);
    ECRM_DISPATCH(direct_for, a, PE != nullptr, st);
}

}  // namespace ecrm
