// Small and medium batches (up to kBucketMaxBatch updates).  What bounds them is not the memory but the number of
// dependent steps: the general path -- a radix sort, the split chains, the apply kernel -- is 13 to 20 launches of 2-5 us,
// and it walks runs of up to 1024 updates with one wavefront.  Here the batch goes through three kernels instead:
//
//   bucket_partition  every tile of the batch is ordered, in arrival order, by bucket -- a hash of the stripe -- and
//                     written out together with the table of where each bucket begins in it; the range check and the
//                     load counts of the tile are done on the way.  No scan over tiles: a bucket is the list of its
//                     pieces in the tiles.  The entries of hot stripes, found in a sample, get buckets of their own.
//   bucket_apply      one workgroup per bucket collects the pieces in LDS, sorts them by (row, position) there and
//                     applies the bucket's stripes.  Hot stripes are split over their columns, which are independent
//                     chains, by workgroups that begin before the buckets'.
//   heavy_stripes     stripes with long runs that were found late, or are too long to be worked off beside the buckets:
//                     split over the columns; of very long ones the runs are cut up as well.
//
// The results are those of the general path: fp64 chains in arrival order, every touched element rounded once.
// Measured against the general path (us a call, D = 128): 26 624 half Zipf 173 -> 49 (to 57 from one
// draw of the keys to the next); 65 536 uniform on 2^14 rows 60 -> 38; 300 007 Zipf, combined rule 325 -> 173.
#include <type_traits>

#include "lists.h"

namespace ecrm {

constexpr int kPartWaves = kPartThreads / kWave;

// ================================================================================================
// partition
// ================================================================================================

struct PartitionArgs {
    const uint64_t *keys;
    u64 *items;                // [n]: tile by tile, row << 32 | position in the batch
    uint16_t *table;           // [tiles][buckets + kHotBuckets + 1]: where each bucket begins in the tile
    uint32_t *tile_cnt;        // [tiles][2S]: load counts of the tile (not for the combined rules)
    uint32_t *tile_state;      // [tiles]: updates that are held back, twice, and one if a key is out of range
    Header *hdr;
    uint32_t n, tiles, buckets, rows, count, D;
    uint32_t clear_sticky, packed;
    Divider dk, dS;
    RecoveryView rv;
};

// sort key of one key of the batch: its row, its stripe; false if it takes no part (out of range, or held back)
__device__ __forceinline__ bool takes_part(const PartitionArgs &a, uint64_t k64, uint32_t &x, uint32_t &g, bool &bad)
{
    x = (uint32_t)k64;
    g = 0;
    bad = !a.packed && k64 >= (uint64_t)a.rows;
    if (bad || held_back(a.rv, x, a.dk, a.dS)) return false;
    g = a.dk.div(x);
    return true;
}

// Stripes that the sample of the batch (bucket_plan.h), the same for every workgroup, holds so often that they are likely
// to have kHotRun updates or more.  Their entries get buckets of their own behind the others, so that neither the sorting
// of a bucket nor the walk of a workgroup sees a hot run; a stripe that the sample misses is found in its bucket.  The
// choice depends on nothing but the sample: every workgroup makes the same one.
constexpr uint32_t kSampleSlots = 2048, kHotCand = 256, kHotSlots = 256;

struct SampleShared {
    uint32_t g[kSampleSlots], c[kSampleSlots];                     // stripe; hits (and, if asked for, a bit << 16 for each of its first 16 entries)
    uint32_t cand_g[kHotCand], cand_c[kHotCand];
};
constexpr uint32_t kHitsMask = 0xFFFFu;
static_assert(kSample <= kHitsMask && kInPlaceEntries <= 16u, "hits and entries in one word");
struct HotShared {
    uint32_t g[kHotSlots], h[kHotSlots];       // open addressing: stripe, its number among the hot ones
    uint32_t n_cand;
};

__device__ __forceinline__ uint32_t find_hot(const PartitionArgs &a, uint32_t n, bool entries, SampleShared &t, HotShared &hot)
{
    const uint32_t tid = threadIdx.x;
    const uint32_t sample = 1u << sample_bits(n), least = hot_hits(n), cap = min(kHotMax, kHotBuckets / a.dk.d);
    for (uint32_t i = tid; i < kSampleSlots; i += kPartThreads) {
        t.g[i] = kNoKey;
        t.c[i] = 0;
    }
    for (uint32_t i = tid; i < kHotSlots; i += kPartThreads) hot.g[i] = kNoKey;
    if (tid == 0) hot.n_cand = 0;
    __syncthreads();
    uint64_t key[kSample / kPartThreads];
#pragma unroll
    for (uint32_t r = 0; r < kSample / kPartThreads; ++r)
        key[r] = r * kPartThreads < sample ? a.keys[sample_position(r * kPartThreads + tid, n)] : 0u;
#pragma unroll
    for (uint32_t r = 0; r < kSample / kPartThreads; ++r) {
        uint32_t x, g;
        bool bad;
        if (r * kPartThreads >= sample || !takes_part(a, key[r], x, g, bad)) continue;
        for (uint32_t s = scramble32(g) & (kSampleSlots - 1u);; s = (s + 1u) & (kSampleSlots - 1u)) {   // at most kSample slots fill
            const uint32_t was = atomicCAS(&t.g[s], kNoKey, g);
            if (was == kNoKey || was == g) {
                const uint32_t j = x - g * a.dk.d;
                atomicAdd(&t.c[s], 1u);
                if (entries && j < kInPlaceEntries) atomicOr(&t.c[s], 0x10000u << j);
                break;
            }
        }
    }
    __syncthreads();
    for (uint32_t i = tid; i < kSampleSlots; i += kPartThreads) {
        if ((t.c[i] & kHitsMask) >= least) {                        // at most kSample / 4 = kHotCand of them
            const uint32_t at = atomicAdd(&hot.n_cand, 1u);
            t.cand_g[at] = t.g[i];
            t.cand_c[at] = t.c[i];
        }
    }
    __syncthreads();
    const uint32_t nc = hot.n_cand;
    if (tid < nc) {                                                 // the cap most frequent, smaller numbers first
        const uint32_t g = t.cand_g[tid], what = t.cand_c[tid], c = what & kHitsMask;
        uint32_t rank = 0;
        for (uint32_t i = 0; i < nc; ++i) {
            const uint32_t ci = t.cand_c[i] & kHitsMask;
            rank += ci > c || (ci == c && t.cand_g[i] < g) ? 1u : 0u;
        }
        if (rank < cap) {
            t.c[rank] = what;                                       // for divide_hot
            uint32_t s = scramble32(g) & (kHotSlots - 1u);
            while (atomicCAS(&hot.g[s], kNoKey, g) != kNoKey) s = (s + 1u) & (kHotSlots - 1u);     // kHotMax < kHotSlots
            hot.h[s] = rank;
        }
    }
    __syncthreads();
    return min(nc, cap);
}

// What is worked off beside the buckets and what is left to heavy_stripes (bucket_plan.h), from what the sample says of the
// hot stripes.  One wave, after find_hot.  All whose size allows it, or none: where some are left, their time comes on top.
// A stripe's time is that of its hits less their standard deviation: the longest of many equal ones looks longer than they are.
__device__ __forceinline__ void divide_hot(const PartitionArgs &a, uint32_t n, uint32_t n_hot, const SampleShared &t, const HotShared &found)
{
    const uint32_t lane = lane_id(), k = a.dk.d, what = lane < n_hot ? t.c[lane] : 0u, hits = what & kHitsMask;
    const uint32_t entries = sampled_entries(hits, (uint32_t)__popc(what >> 16), k), updates = sampled_updates(hits, n);
    uint32_t all = updates;
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) all += __shfl_xor(all, d, kWave);
    const HotStripe longest{from_lane(updates, 0), from_lane(entries, 0)}, mine{sampled_updates(hits - square_root(hits), n), entries};
    const BucketLimits lim = bucket_limits(n, k, a.D);
    const bool fits = lane < n_hot && in_place_size(lim, k, updates);
    const u64 slow = __ballot(fits && !in_place_time(lim, a.D, n_hot, n - min(all, n), longest, mine));
    const u64 here = slow ? 0ull : __ballot(fits);
    const u64 left = __ballot(lane < n_hot && updates >= hot_least(lim, k, found.n_cand)) & ~here;
    if (lane == 0) {
        a.hdr->hot_here = here;
        a.hdr->heavy_run = left && a.D <= 128u ? heavy_run_beside(n) : heavy_run(n);
    }
}

// Bound by its chain of dependent steps (keys, ranks, scan, write), not by its 16 bytes per update; the ranks are
// those of the sort's scatter kernel -- equal buckets of a wave are matched with ballots -- with one 16-bit counter per
// wave and bucket, the eight of a bucket side by side in LDS.
template <int IPT>
__global__ __launch_bounds__(kPartThreads) void bucket_partition_kernel(PartitionArgs a)
{
    constexpr uint32_t kTile = kPartThreads * IPT;
    __shared__ __align__(16) uint16_t s_cnt[kMaxBuckets + kHotBuckets][kPartWaves];
    __shared__ HotShared s_hot;
    __shared__ uint32_t s_srv[2 * kBucketMaxServers];
    __shared__ uint32_t s_wave[kPartWaves], s_held;
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid / kWave, tile = blockIdx.x;
    const uint32_t n = a.packed ? min(a.n, a.hdr->buf_count) : a.n;       // a replay: everything that is waiting now
    const uint32_t S = a.dS.d, tile0 = tile * kTile;
    static_assert(sizeof(SampleShared) <= sizeof(s_cnt), "the sample is counted where the buckets are, before them");
    SampleShared &sample = *(SampleShared *)&s_cnt[0][0];
    const uint32_t n_hot = n >= kSample * 4u ? find_hot(a, n, tile == a.tiles, sample, s_hot) : 0u;
    if (tile == a.tiles) {                                                // no tile: one workgroup more, beside the others
        if (wave == 0) divide_hot(a, n, n_hot, sample, s_hot);
        return;
    }
    // a replay's buckets are those of what is waiting, not of the buffer that holds it: 4096 workgroups for 20 000 updates
    const uint32_t ordinary = a.packed ? bucket_count(n) : a.buckets;
    // ... and some of the plan's stay empty where hot stripes are worked off beside them
    const bool beside = !a.packed && !a.rv.active && beside_pays(a.dk.d, a.D);
    const uint32_t used = beside ? buckets_beside(ordinary, n_hot, a.D) : ordinary;
    const uint32_t B = ordinary + kHotBuckets;                            // buckets in the table; the last are the hot entries'
    for (uint32_t i = tid; i < B; i += kPartThreads) *(ulonglong2 *)s_cnt[i] = ulonglong2{0, 0};
    for (uint32_t i = tid; i < 2 * S; i += kPartThreads) s_srv[i] = 0;
    if (tid == 0) s_held = 0;
    __syncthreads();

    uint32_t held = 0, row[IPT], dig[IPT], rank[IPT];
    bool in[IPT], bad = false;
#pragma unroll
    for (int r = 0; r < IPT; ++r) {
        const uint32_t i = tile0 + wave * (kWave * IPT) + r * kWave + lane;
        row[r] = dig[r] = 0;
        in[r] = false;
        if (i < n) {
            uint32_t x, g;
            bool out;
            in[r] = takes_part(a, a.keys[i], x, g, out);
            bad |= out;
            held += !in[r] && !out ? 1u : 0u;
            if (in[r]) {
                const uint32_t j = x - g * a.dk.d;
                row[r] = x;
                dig[r] = bucket_of(g, used);
                if (n_hot) {
                    for (uint32_t s = scramble32(g) & (kHotSlots - 1u); s_hot.g[s] != kNoKey; s = (s + 1u) & (kHotSlots - 1u)) {
                        if (s_hot.g[s] == g) {
                            dig[r] = ordinary + s_hot.h[s] * a.dk.d + j;
                            break;
                        }
                    }
                }
                if (a.count) {
                    atomicAdd(&s_srv[a.dS.mod(g + 1 + j)], 1u);
                    atomicAdd(&s_srv[S + a.dS.mod(g)], 1u);
                }
            }
        }
    }
    if (held) atomicAdd(&s_held, held);
    const int bits = 32 - __builtin_clz(n_hot ? B - 1u : max(ordinary - 1u, 1u));
#pragma unroll
    for (int r = 0; r < IPT; ++r) {
        u64 peers = __ballot(in[r]);
        for (int b = 0; b < bits; ++b) {
            const bool bit = (dig[r] >> b) & 1u;
            const u64 bal = __ballot(bit);
            peers &= bit ? bal : ~bal;
        }
        const uint32_t below = (uint32_t)__popcll(peers & bits_below(lane));
        const uint32_t old = s_cnt[dig[r]][wave];
        __builtin_amdgcn_wave_barrier();
        if (in[r] && below == 0) s_cnt[dig[r]][wave] = (uint16_t)(old + (uint32_t)__popcll(peers));
        __builtin_amdgcn_wave_barrier();
        rank[r] = old + below;
    }
    bad = __syncthreads_or(bad);

    uint16_t *out = a.table + (size_t)tile * (B + 1);
    uint32_t carry = 0;
    for (uint32_t d0 = 0; d0 < B; d0 += kPartThreads) {
        const uint32_t d = d0 + tid;
        uint32_t c[kPartWaves], tot = 0;
#pragma unroll
        for (int w = 0; w < kPartWaves; ++w) {
            c[w] = d < B ? s_cnt[d][w] : 0u;
            tot += c[w];
        }
        uint32_t all;
        uint32_t at = carry + bucket_excl_scan<kPartWaves>(tot, s_wave, all);
        carry += all;
        if (d < B) {
            out[d] = (uint16_t)at;
#pragma unroll
            for (int w = 0; w < kPartWaves; ++w) {
                s_cnt[d][w] = (uint16_t)at;
                at += c[w];
            }
        }
    }
    if (tid == 0) {
        out[B] = (uint16_t)carry;
        a.tile_state[tile] = 2u * s_held + (bad ? 1u : 0u);
    }
    if (a.count)
        for (uint32_t i = tid; i < 2 * S; i += kPartThreads) a.tile_cnt[(size_t)tile * 2 * S + i] = s_srv[i];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < IPT; ++r) {
        const uint32_t i = tile0 + wave * (kWave * IPT) + r * kWave + lane;
        if (in[r]) a.items[tile0 + s_cnt[dig[r]][wave] + rank[r]] = ((u64)row[r] << 32) | i;
    }
    // the header of the call: no other workgroup of this launch touches it (a replay reads buf_count only)
    if (tile == 0 && tid == 0) {
        begin_batch(a.hdr, n, a.clear_sticky != 0);
        a.hdr->n_hot = n >= kSample * 4u ? s_hot.n_cand : 0u;
    }
}

// ================================================================================================
// one workgroup per bucket
// ================================================================================================

struct BucketArgs : RowArgs {
    const uint64_t *keys;        // the batch: the caller's keys, or the list entries of a replay (packed)
    const u64 *items;
    u64 *tmp, *dense;            // [n] each: an oversized bucket's items in arrival order; its heavy stripes', sorted
    const uint16_t *table;
    const uint32_t *tile_cnt, *tile_state;
    uint32_t *heavy;             // [2 * (n / kHeavyRunMin + 64)]: start in `dense`, number of updates
    SplitScratch split;          // of stripes whose runs are cut up
    Header *hdr;
    u64 *load_data, *load_parity;
    uint32_t *rejected;          // null, or where the caller wants to read whether the batch was rejected
    uint32_t n, tile, tiles, buckets, packed;
    uint32_t holding;            // a recovery is in progress: the header follows what hold_tiles did
    BucketLimits lim;
};

// A replay has as many updates as were waiting, not as many as the buffer holds: the partition's plan.
__device__ __forceinline__ void plan_replay(BucketArgs &a)
{
    if (!a.packed) return;
    a.n = min(a.n, a.hdr->n_batch);
    a.tiles = (a.n + a.tile - 1u) / a.tile;
    a.buckets = bucket_count(a.n);
    a.lim = bucket_limits(a.n, a.geo.k, a.geo.D);
}

// The kernel's arguments, read once more: what is needed on rare paths only is not kept in scalar registers across the walk,
// which needs all of them (a hundred were spilled).  They are read from where the kernel's first argument lies, so it has to be the
// only one (bucket_apply_for).  The pointers are read as pointers to device memory: after a flat access
// the compiler has the walk wait for all of its loads.
template <typename T>
__device__ __forceinline__ void read_global(T *&p, const __attribute__((address_space(4))) char *from)
{
    typedef __attribute__((address_space(1))) T *global;
    p = (T *)*(const __attribute__((address_space(4))) global *)from;
}
__device__ __forceinline__ BucketArgs args_again()
{
    typedef __attribute__((address_space(4))) const char byte;
    typedef __attribute__((address_space(4))) const u64 word;
    static_assert(sizeof(BucketArgs) % sizeof(u64) == 0 && alignof(BucketArgs) == alignof(u64), "copied word by word");
    byte *p = (byte *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    u64 w[sizeof(BucketArgs) / sizeof(u64)];
#pragma unroll
    for (uint32_t i = 0; i < sizeof(BucketArgs) / sizeof(u64); ++i) w[i] = ((word *)p)[i];
    BucketArgs a;
    __builtin_memcpy(&a, w, sizeof(a));
    auto again = [&](auto &field) { read_global(field, p + ((const char *)&field - (const char *)&a)); };
    again(a.E); again(a.A); again(a.PE); again(a.PA); again(a.grads); again(a.keys); again(a.items); again(a.tmp);
    again(a.dense); again(a.table); again(a.tile_cnt); again(a.tile_state); again(a.heavy); again(a.split.run);
    again(a.split.tiles); again(a.split.segment_run); again(a.split.summed); again(a.split.arrived); again(a.split.sums);
    again(a.split.steps); again(a.hdr); again(a.load_data); again(a.load_parity);
    plan_replay(a);
    return a;
}

// gradient row of an item, from its position in the batch
__device__ __forceinline__ u64 resolved(const BucketArgs &a, u64 it)
{
    return a.packed ? (it & 0xFFFFFFFF00000000ull) | (a.keys[(uint32_t)it] >> 32) : it;
}

// One more stripe for heavy_stripes, at base + at0 in `dense` (one thread).  Every such stripe has at least kHeavyRunMin
// updates, or is one of the at most kHotMax that the sample found: there is room in the list.
constexpr uint32_t kCounted = 0x80000000u;  // flag beside the number: the combined rules' load is counted already
__device__ __forceinline__ void list_heavy(const BucketArgs &a, uint32_t &dense_used, uint32_t base, uint32_t at0, uint32_t count,
                                           bool counted)
{
    const uint32_t i = atomicAdd(&a.hdr->n_heavy, 1u);
    a.heavy[2 * i] = base + at0;
    a.heavy[2 * i + 1] = count | (counted ? kCounted : 0u);
    dense_used = at0 + count;
}

constexpr uint32_t kStripeSlots = 1024;     // LDS table of an oversized bucket's stripes
constexpr uint32_t kStripeFill = 640;       // ... and how many it may hold
constexpr uint32_t kHeavySlots = 16;

struct BucketShared {
    __align__(16) u64 item[kBucketCap];
    union {
        __align__(16) u64 tmp[kBucketCap];                     // of the sort, and sums of walk_long_stripe
        struct { uint32_t tab_g[kStripeSlots], tab_c[kStripeSlots]; };     // of an oversized bucket, before it
        ExchangeOf<kBucketWaves> ex[2];                        // of a hot stripe
    };
    union {
        FewRows few;                                           // before the list is walked
        ListShared<kBucketCap> list;
    };
    uint32_t pref[kMaxTiles + 1], start[kMaxTiles], wave[kBucketWaves];
    uint32_t hv[kHeavySlots], hv_n, fill, light, n_light, over;
    uint32_t member[kBucketWaves][64];
    uint32_t dense_used;
};

__device__ __forceinline__ uint32_t stripe_slot(const uint32_t *tab_g, uint32_t g)      // g is in the table
{
    uint32_t s = (g * 0x85EBCA77u) >> 22;
    while (tab_g[s] != g) s = (s + 1u) & (kStripeSlots - 1u);
    return s;
}

// where the q-th item, in arrival order, of a bucket lies in a.items: pref are its items in earlier tiles, start its places
__device__ __forceinline__ uint32_t place_of(const uint32_t *pref, const uint32_t *start, uint32_t tiles, uint32_t q)
{
    uint32_t lo = 0, hi = tiles;                                    // pref[lo] <= q < pref[hi]
    while (hi - lo > 1u) {
        const uint32_t mid = (lo + hi) / 2u;
        if (pref[mid] <= q) lo = mid; else hi = mid;
    }
    return start[lo] + (q - pref[lo]);
}

// A bucket with more items than LDS takes: hot stripes.  Its items are first laid out in arrival order in tmp; then,
// for one part of the stripes after the other (by the low bits of the mix, split until a part fits), the stripes are
// counted in an LDS table, the light ones are collected, sorted and applied like any bucket, and the heavy ones --
// heavy_stripe(k) updates or more -- are written to `dense`, entry by entry in arrival order, for heavy_stripes.  A part of a
// single stripe always fits, so the splitting ends.  Uniform over the workgroup.  Every pass over the items keeps
// kAhead loads of a thread in flight (one at a time, a bucket of 14 000 items took 130 us).
constexpr int kAhead = 4;

// the bucket's items in arrival order; RESOLVE: with their gradient rows in place of their positions.  A wave takes whole
// pieces, kCopyAhead of them at a time: each step is a trip to memory.
template <bool RESOLVE>
__device__ __forceinline__ void copy_bucket(const BucketArgs &a, const BucketShared &sh, u64 *to)
{
    constexpr uint32_t kCopyAhead = 8;
    const uint32_t lane = lane_id();
    for (uint32_t t0 = uniform(threadIdx.x / kWave) * kCopyAhead; t0 < a.tiles; t0 += kBucketWaves * kCopyAhead) {
        uint32_t longest = 0;
#pragma unroll
        for (uint32_t u = 0; u < kCopyAhead; ++u) {
            const uint32_t t = min(t0 + u, a.tiles - 1u);
            longest = max(longest, sh.pref[t + 1] - sh.pref[t]);
        }
        for (uint32_t c = lane; c - lane < longest; c += kWave) {
            u64 it[kCopyAhead];
#pragma unroll
            for (uint32_t u = 0; u < kCopyAhead; ++u) {
                const uint32_t t = min(t0 + u, a.tiles - 1u);
                it[u] = c < sh.pref[t + 1] - sh.pref[t] ? a.items[sh.start[t] + c] : 0ull;
            }
#pragma unroll
            for (uint32_t u = 0; u < kCopyAhead; ++u) {
                const uint32_t t = t0 + u;
                if (t < a.tiles && c < sh.pref[t + 1] - sh.pref[t]) to[sh.pref[t] + c] = RESOLVE ? resolved(a, it[u]) : it[u];
            }
        }
    }
}

__device__ __forceinline__ void oversized_begin(const BucketArgs &a, BucketShared &sh, uint32_t base)
{
    copy_bucket<false>(a, sh, a.tmp + base);
    if (threadIdx.x == 0) sh.dense_used = 0;
    __threadfence_block();
    __syncthreads();
}

// f(item) for the items [lo, hi) of tmp, `lane` of `width` taking every width-th; positions past hi: f(~0)
template <typename F>
__device__ __forceinline__ void stream_items(const u64 *tmp, uint32_t lo, uint32_t hi, uint32_t lane, uint32_t width, F f)
{
    for (uint32_t q0 = lo; q0 < hi; q0 += kAhead * width) {
        u64 it[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const uint32_t q = q0 + u * width + lane;
            it[u] = q < hi ? tmp[q] : ~0ull;
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) f(it[u]);
    }
}

// The parts still to come: `part` are the low `depth` bits of the next one; depth < 0: none is left.
struct PartWalk {
    uint32_t part;
    int depth;
};

// One part: its heavy stripes go to `dense`, its light ones' items to LDS, not sorted yet; returns how many they are.
__device__ __forceinline__ uint32_t oversized_part(const BucketArgs &a, BucketShared &sh, uint32_t m, uint32_t base,
                                                   PartWalk &walk)
{
    const uint32_t tid = threadIdx.x, lane = lane_id(), w = uniform(tid / kWave), k = a.geo.k;
    const Divider dk = a.geo.dk;
    const u64 *tmp = a.tmp + base;
    u64 *dense = a.dense + base;
    const uint32_t heavy = heavy_stripe(k);
    uint32_t part = walk.part, mask;
    int depth = walk.depth;
    for (;;) {
        mask = depth >= 32 ? ~0u : (1u << depth) - 1u;
        // ---- count the part's stripes
        for (uint32_t i = tid; i < kStripeSlots; i += kBucketThreads) {
            sh.tab_g[i] = kNoKey;
            sh.tab_c[i] = 0;
        }
        if (tid == 0) sh.fill = sh.light = sh.n_light = sh.over = sh.hv_n = 0;
        __syncthreads();
        auto *over = (volatile __attribute__((address_space(3))) uint32_t *)&sh.over;
        stream_items(tmp, 0, m, tid, kBucketThreads, [&](u64 it) {
            const uint32_t g = dk.div(item_row(it));
            // one lane for all of the wave's items of its stripe: a hot stripe's counter, updated by every lane, is
            // what this pass would wait for
            bool in = it != ~0ull && (scramble32(g) & mask) == part;
            uint32_t c = 0;
            for (u64 todo = __ballot(in); todo;) {
                const u64 same = __ballot(in && g == from_lane(g, lowest_bit(todo)));
                if (lane == lowest_bit(todo)) c = (uint32_t)__popcll(same);
                todo &= ~same;
            }
            if (c == 0 || *over) return;
            uint32_t s = (g * 0x85EBCA77u) >> 22, tries = 0;
            for (; tries < kStripeSlots; ++tries) {                 // bounded: a full table means the part is split
                const uint32_t was = atomicCAS(&sh.tab_g[s], kNoKey, g);
                if (was == kNoKey && atomicAdd(&sh.fill, 1u) >= kStripeFill) *over = 1;
                if (was == kNoKey || was == g) break;
                s = (s + 1u) & (kStripeSlots - 1u);
            }
            if (tries < kStripeSlots) atomicAdd(&sh.tab_c[s], c);
            else *over = 1;
        });
        __syncthreads();
        if (!sh.over) {
            for (uint32_t s = tid; s < kStripeSlots; s += kBucketThreads) {
                const uint32_t c = sh.tab_c[s];
                if (c >= heavy) {
                    const uint32_t i = atomicAdd(&sh.hv_n, 1u);
                    if (i < kHeavySlots) sh.hv[i] = s;
                } else if (c) {
                    atomicAdd(&sh.light, c);
                }
            }
        }
        __syncthreads();
        const bool split = sh.over || sh.hv_n > kHeavySlots || sh.light > kBucketCap;
        __syncthreads();
        if (!split) break;                                          // ends: a part of one stripe fits
        ++depth;
    }
    // ---- the light stripes
    const uint32_t light = uniform(sh.light), nh = uniform(sh.hv_n);
    if (light)
        stream_items(tmp, 0, m, tid, kBucketThreads, [&](u64 it) {
            const uint32_t g = dk.div(item_row(it));
            if (it == ~0ull || (scramble32(g) & mask) != part) return;
            if (sh.tab_c[stripe_slot(sh.tab_g, g)] < heavy) sh.item[atomicAdd(&sh.n_light, 1u)] = it;
        });
    // ---- the heavy ones: a stable partition by member, every wave a contiguous quarter of the items
    const uint32_t quarter = (m + kBucketWaves - 1) / kBucketWaves, q_lo = min(w * quarter, m), q_hi = min(q_lo + quarter, m);
    for (uint32_t h = 0; h < nh; ++h) {
        const uint32_t slot = uniform(sh.hv[h]), g = uniform(sh.tab_g[slot]), c = uniform(sh.tab_c[slot]);
        for (uint32_t j = tid; j < kBucketWaves * 64u; j += kBucketThreads) (&sh.member[0][0])[j] = 0;
        __syncthreads();
        stream_items(tmp, q_lo, q_hi, lane, kWave, [&](u64 it) {
            const uint32_t x = item_row(it);
            const bool in = it != ~0ull && dk.div(x) == g;
            for (u64 todo = __ballot(in); todo;) {                  // at most k rounds
                const uint32_t who = lowest_bit(todo);
                const u64 same = __ballot(in && x == from_lane(x, who));
                if (lane == who) sh.member[w][x - g * k] += (uint32_t)__popcll(same);      // the wave's own counter
                todo &= ~same;
            }
        });
        __syncthreads();
        const uint32_t at0 = uniform(sh.dense_used);
        if (w == 0) {                                               // lane j: where member j's updates begin, wave by wave
            uint32_t cnt[kBucketWaves], all = 0;
#pragma unroll
            for (int v = 0; v < kBucketWaves; ++v) {
                cnt[v] = sh.member[v][lane];
                all += cnt[v];
            }
            uint32_t incl = all;
#pragma unroll
            for (int d = 1; d < kWave; d <<= 1) {
                const uint32_t t = __shfl_up(incl, d, kWave);
                if (lane >= (uint32_t)d) incl += t;
            }
            uint32_t at = at0 + incl - all;
#pragma unroll
            for (int v = 0; v < kBucketWaves; ++v) {
                sh.member[v][lane] = at;
                at += cnt[v];
            }
        }
        __syncthreads();
        stream_items(tmp, q_lo, q_hi, lane, kWave, [&](u64 it) {
            const uint32_t x = item_row(it);
            const bool mine = it != ~0ull && dk.div(x) == g;
            const uint32_t j = mine ? x - g * k : 0u;
            u64 peers = __ballot(mine);
#pragma unroll
            for (int b = 0; b < 6; ++b) {
                const bool bit = (j >> b) & 1u;
                const u64 bal = __ballot(bit);
                peers &= bit ? bal : ~bal;
            }
            const uint32_t at = sh.member[w][j], below = (uint32_t)__popcll(peers & bits_below(lane));
            __builtin_amdgcn_wave_barrier();
            if (mine) {
                dense[at + below] = resolved(a, it);
                if (below == 0) sh.member[w][j] = at + (uint32_t)__popcll(peers);
            }
            __builtin_amdgcn_wave_barrier();
        });
        __syncthreads();                                            // every wave has taken at0
        if (tid == 0) list_heavy(a, sh.dense_used, base, at0, c, false);
        __syncthreads();
    }
    // ---- next part: the parts are the leaves of a binary tree over the low bits, left to right
    while (depth > 0 && ((part >> (depth - 1)) & 1u)) {
        part &= ~(1u << (depth - 1));
        --depth;
    }
    if (depth > 0) part |= 1u << (depth - 1);
    walk.part = part;
    walk.depth = depth > 0 ? depth : -1;
    __syncthreads();
    return light;
}

// One entry, the r-th hot bucket, of a stripe of split_stripe updates or more: its updates are left where the partition put
// them, and described -- how many, where each tile's lie -- and cut into segments for heavy_stripes.
__device__ __forceinline__ void split_run(const BucketArgs &a, BucketShared &sh, uint32_t r, uint32_t from, uint32_t len)
{
    const uint32_t tid = threadIdx.x, ncg = (a.geo.D + kHeavyCols - 1) / kHeavyCols;
    uint32_t m;
    const uint32_t at = bucket_excl_scan(len, sh.wave, m);
    const uint32_t segs = (m + kSplitSegment - 1) / kSplitSegment;
    if (tid == 0) {
        sh.fill = segs ? atomicAdd(&a.hdr->n_segments, segs) : 0u;
        a.split.run[r] = SplitRun{sh.fill, m};
    }
    uint32_t *pref = a.split.tiles + (size_t)r * kSplitTileWords, *start = pref + kMaxTiles + 1;
    if (tid < a.tiles) {
        pref[tid] = at;
        start[tid] = from;
    }
    if (tid == 0) pref[a.tiles] = m;
    __syncthreads();
    const uint32_t first = sh.fill;
    for (uint32_t i = tid; i < segs; i += kBucketThreads) a.split.segment_run[first + i] = r;
    for (uint32_t i = tid; i < segs * ncg; i += kBucketThreads) a.split.summed[(size_t)first * ncg + i] = 0;
    if (r % a.geo.k == 0)
        for (uint32_t i = tid; i < ncg; i += kBucketThreads) a.split.arrived[r / a.geo.k * ncg + i] = 0;
}

// ---- hot stripes -----------------------------------------------------------------------------------
// The stripes that the sample took for hot, numbered as they are ranked.  The first kHotMax workgroups look after one each,
// should it be short after all; the others of the hot buckets' kHotBuckets hand on what is left to heavy_stripes, and take
// (stripe, 16 columns) jobs of the rest, so that what takes long begins first and beside everything else: as a launch of its own
// behind this one it was 7 to 11 us of a call.  Which way they go is the partition's choice (divide_hot).

// one entry's updates, or a whole stripe's: how many, where each tile's lie
struct HotSpan { uint32_t from, len; };
__device__ __forceinline__ HotSpan hot_span(const BucketArgs &a, uint32_t first_bucket, uint32_t buckets)
{
    HotSpan s{0, 0};
    if (threadIdx.x < a.tiles) {
        const uint16_t *row = a.table + (size_t)threadIdx.x * (a.buckets + kHotBuckets + 1) + first_bucket;
        s.from = threadIdx.x * a.tile + row[0];
        s.len = (uint32_t)row[buckets] - row[0];
    }
    return s;
}

// The stripe that a workgroup of the hot buckets looks at first: the one it looks after, or that of the first entry that it may
// have to hand on.  Asked for before it is known how many there are, so it has to lie inside the hot buckets.
__device__ __forceinline__ uint32_t first_hot_stripe(const Geometry &geo)
{
    return blockIdx.x < kHotMax ? min(blockIdx.x, kHotBuckets / geo.k - 1u) : geo.dk.div(blockIdx.x - kHotMax);
}
static_assert(kHotMax >= 64u, "the stripe of the last workgroup's entry ends with the hot buckets");

// 16 columns of hot stripe h, whose updates are left where the partition put them.  As in long_runs.h, with T updates to a
// group of eight lanes and 32 groups: 256 updates a round.
template <int MODE, bool PARITY>
__device__ __forceinline__ void hot_job(const BucketArgs &a, BucketShared &sh, uint32_t h, uint32_t cg)
{
    constexpr int T = 8;
    constexpr uint32_t kRound = kBucketThreads / 8 * T;
    const uint32_t D = a.geo.D, k = a.geo.k, tid = threadIdx.x, lane = lane_id(), w = uniform(tid / kWave);
    const uint32_t col_lane = lane & 7u, sub = w * 8u + lane / 8u, col = cg * kHeavyCols + 2u * col_lane;
    const bool live = col < D;                                      // D is a multiple of 4: both columns or none
    const RuleParams rp = rule_params(a.geo);
    uint32_t g = kNoKey, buf = 0;
    D2 pe = D2{-0.0, -0.0}, pa = D2{-0.0, -0.0};                    // the differences; the neutral summand
    for (uint32_t j = 0; j < k; ++j) {
        const HotSpan s = hot_span(a, a.buckets + h * k + j, 1);
        uint32_t L;
        const uint32_t at = bucket_excl_scan(s.len, sh.wave, L);
        if (L == 0) continue;
        if (tid < a.tiles) {
            sh.pref[tid] = at;
            sh.start[tid] = s.from;
        }
        if (tid == 0) sh.pref[a.tiles] = L;
        __syncthreads();
        // the lanes of a group look up an update each (past the run's end: the last one)
        auto look = [&](uint32_t r0) {
            return resolved(a, a.items[place_of(sh.pref, sh.start, a.tiles, min(r0 + sub * T + col_lane, L - 1u))]);
        };
        float2 gr[T], nx[T];
        auto rows = [&](uint32_t idx, uint32_t r0) {
#pragma unroll
            for (int u = 0; u < T; ++u) {
                const uint32_t i = __shfl(idx, (int)((lane & 56u) + u), kWave);
                nx[u] = float2{0, 0};
                if (live && r0 + sub * T + u < L) nx[u] = *(const float2 *)(a.grads + (size_t)i * D + col);
            }
        };
        const u64 it = look(0);
        uint32_t idx = (uint32_t)it;
        const uint32_t x = uniform(item_row(it));
        rows(idx, 0);
        idx = (uint32_t)look(kRound);
        g = a.geo.dk.div(x);
        float2 a0 = float2{0, 0};
        if (live) a0 = *(const float2 *)(a.A + (size_t)x * D + col);
        D2 state = start2<MODE>(widen2(a0)), acc = D2{0, 0};
        for (uint32_t r0 = 0; r0 < L; r0 += kRound) {
            const uint32_t off = r0 + sub * T, cnt = off < L ? min((uint32_t)T, L - off) : 0u;
#pragma unroll
            for (int u = 0; u < T; ++u) gr[u] = nx[u];
            if (r0 + kRound < L) {
                rows(idx, r0 + kRound);
                idx = (uint32_t)look(r0 + 2u * kRound);
            }
            if (Rule<MODE>::combine) {                              // a sum: nothing to exchange before the run's end
#pragma unroll
                for (int u = 0; u < T; ++u) {                       // zeros past the end of the run
                    acc.x += (double)gr[u].x;
                    acc.y += (double)gr[u].y;
                }
                continue;
            }
            double ed;
            const D2 ex = heavy_sums<MODE>(gr, cnt, rp, sh.ex[buf], w, ed);
            __syncthreads();
            D2 mine = heavy_fold<MODE>(state, sh.ex[buf], w, ex, ed);
#pragma unroll
            for (int u = 0; u < T; ++u) asm volatile("" : "+v"(gr[u].x), "+v"(gr[u].y));     // widened once more (walk_columns)
#pragma unroll
            for (int u = 0; u < T; ++u) {
                if ((uint32_t)u < cnt) item2<MODE>(mine, acc, gr[u], rp);
            }
            buf ^= 1u;                                              // a half is written again only behind the other's barrier
        }
        acc = heavy_total(acc, sh.ex[buf], w);
        buf ^= 1u;
        if (Rule<MODE>::combine) {
            state = acc;
            acc = D2{0, 0};
        }
        const D2 a64 = widen2(a0);
        finish2<MODE>(state, acc, a64, rp);
        if (live && sub == 0) {
            float2 *e = (float2 *)(a.E + (size_t)x * D + col);
            const D2 e64 = widen2(*e);
            *e = narrow2(D2{e64.x - acc.x, e64.y - acc.y});
            *(float2 *)(a.A + (size_t)x * D + col) = narrow2(state);
        }
        pe.x -= acc.x;
        pe.y -= acc.y;
        pa.x += state.x - a64.x;
        pa.y += state.y - a64.y;
        if (cg == 0 && tid == 0) {
            if (L > kLongRun) {                                     // reported by ecrm_batch_stats
                atomicAdd(&a.hdr->n_long, 1u);
                atomicAdd(&a.hdr->n_long_items, (u64)L);
            }
            if (Rule<MODE>::combine) {
                atomicAdd(&a.load_data[a.geo.dS.mod(g + 1 + (x - g * k))], 1ull);
                if (a.load_parity) atomicAdd(&a.load_parity[a.geo.dS.mod(g)], 1ull);
            }
        }
        __syncthreads();                                            // sh.pref and sh.start are free for the next entry
    }
    if (PARITY && live && sub == 0 && g != kNoKey) {
        float2 *to = (float2 *)(a.PE + (size_t)g * D + col), *state = (float2 *)(a.PA + (size_t)g * D + col);
        const D2 pe64 = widen2(*to), pa64 = widen2(*state);
        *to = narrow2(D2{pe64.x + pe.x, pe64.y + pe.y});
        *state = narrow2(D2{pa64.x + pa.x, pa64.y + pa.y});
    }
}

// What a workgroup of the hot buckets has to do; true: it goes on with the stripe as an ordinary bucket.  s: first_hot_stripe,
// e: the entry of the same number as the workgroup.
template <int MODE, bool PARITY>
__device__ __forceinline__ bool hot_block(const BucketArgs &a, BucketShared &sh, uint32_t n_hot, u64 here, HotSpan s, HotSpan e)
{
    const uint32_t k = a.geo.k, tid = threadIdx.x, ncg = (a.geo.D + kHeavyCols - 1) / kHeavyCols;
    const uint32_t hot = min(n_hot, min(kHotMax, kHotBuckets / k));
    // no stripe, or one that is not as long as the sample made it look: its entries' buckets lie side by side in every tile,
    // so a workgroup takes them as one ordinary bucket
    const uint32_t least = hot_least(a.lim, k, n_hot);
    if (blockIdx.x < kHotMax) {
        if (blockIdx.x >= hot) return false;
        uint32_t m;
        bucket_excl_scan(s.len, sh.wave, m);
        return m < least;
    }
    constexpr uint32_t kWorkers = kHotWorkers;
    const uint32_t worker = blockIdx.x - kHotMax;
    // Left to heavy_stripes: the entries of the longest are described to it, the others copied, in arrival order, by all of
    // these workgroups alike (by those of the stripe's first columns, 24 of the 192 did all of it with four entries of 512
    // floats: 2^18 updates on 256 such rows 545 us, now 375).
    for (uint32_t q = worker; q < hot * k; q += kWorkers) {
        const uint32_t h = a.geo.dk.div(q), j = q - h * k;
        if (q != worker) {
            s = hot_span(a, a.buckets + h * k, k);
            e = hot_span(a, a.buckets + q, 1);
        }
        uint32_t m;
        bucket_excl_scan(s.len, sh.wave, m);
        if (m < least || (((here >> h) & 1u) && in_place_size(a.lim, k, m))) continue;
        if (m >= a.lim.split_stripe) {
            split_run(a, sh, q, e.from, e.len);
            __syncthreads();                                        // sh.fill
            continue;
        }
        uint32_t L, start, begin;
        const uint32_t at = bucket_excl_scan(e.len, sh.wave, L);
        bucket_excl_scan(tid < a.tiles ? e.from - tid * a.tile : 0u, sh.wave, start);
        if (j == 0) {
            bucket_excl_scan(tid < a.tiles ? s.from - tid * a.tile : 0u, sh.wave, begin);
            if (tid == 0) list_heavy(a, sh.dense_used, begin, 0, m, false);
        }
        if (tid < a.tiles) {
            sh.pref[tid] = at;
            sh.start[tid] = e.from;
        }
        if (tid == 0) sh.pref[a.tiles] = L;
        __syncthreads();
        copy_bucket<true>(a, sh, a.dense + start);
        __syncthreads();
    }
    for (uint32_t job = worker; job < hot * ncg; job += kWorkers) {
        const uint32_t h = job / ncg;
        if (!((here >> h) & 1u)) continue;
        uint32_t m;
        bucket_excl_scan(hot_span(a, a.buckets + h * k, k).len, sh.wave, m);
        if (m >= least && in_place_size(a.lim, k, m)) hot_job<MODE, PARITY>(a, sh, h, job % ncg);
    }
    return false;
}

static_assert(sizeof(BucketShared::tmp) >= (kBucketWaves + 2) * 2 * 128 * sizeof(double), "walk_long_stripe's sums for NC = 2");

template <int NC, int MODE, bool PARITY, bool CUT>
__global__ __launch_bounds__(kBucketThreads, NC == 1 ? 4 : 3) void bucket_apply_kernel(BucketArgs a)
{
    __shared__ BucketShared sh;
    plan_replay(a);
    if (blockIdx.x >= a.buckets + kHotBuckets) return;
    const uint32_t tid = threadIdx.x, B = a.buckets + kHotBuckets, S = a.geo.S;
    // the hot stripes first: what takes longest must not begin last
    const bool of_hot = blockIdx.x < kHotBuckets;
    const uint32_t b = of_hot ? kNoKey : blockIdx.x - kHotBuckets;
    bool key_bad = false;
    uint32_t from = 0, len = 0, entry_from = 0, entry_len = 0;
    if (tid < a.tiles) {
        key_bad = (a.tile_state[tid] & 1u) != 0;
        const uint32_t first = of_hot ? a.buckets + first_hot_stripe(a.geo) * a.geo.k : b, buckets = of_hot ? a.geo.k : 1u;
        const uint16_t *row = a.table + (size_t)tid * (B + 1);
        if (of_hot) {
            const uint32_t entry = a.buckets + (blockIdx.x < kHotMax ? 0u : blockIdx.x - kHotMax);
            entry_from = tid * a.tile + row[entry];
            entry_len = (uint32_t)row[entry + 1u] - row[entry];
        }
        from = tid * a.tile + row[first];
        len = (uint32_t)row[first + buckets] - row[first];
    }
    const uint32_t n_hot = a.hdr->n_hot, heavy_run = a.hdr->heavy_run;
    const u64 here = a.hdr->hot_here;
    const bool many = n_hot > kManyHot;                             // long stripes
    const bool full = a.hdr->batch_bad != 0;                        // the recovery buffer could not take its part
    key_bad = __syncthreads_or(key_bad);
    if (b == 0 && tid == 0 && a.rejected) *a.rejected = key_bad || full ? 1u : 0u;
    if (key_bad || full) {
        if (b == 0 && tid == 0 && key_bad) {
            a.hdr->batch_bad = 1;
            atomicOr(&a.hdr->err_sticky, 1u);
        }
        return;
    }
    if (of_hot && !hot_block<MODE, PARITY>(a, sh, n_hot, here, HotSpan{from, len}, HotSpan{entry_from, entry_len})) return;
    uint32_t m;
    const uint32_t at = bucket_excl_scan(len, sh.wave, m);
    if (!Rule<MODE>::combine && b == 0) {                           // the batch is valid: publish its per-server counts
        for (uint32_t i = tid; i < 2 * S; i += kBucketThreads) sh.list.srv[i] = 0;
        __syncthreads();
        for (uint32_t i = tid; i < a.tiles * 2 * S; i += kBucketThreads) {
            const uint32_t c = a.tile_cnt[i];
            if (c) atomicAdd(&sh.list.srv[i % (2 * S)], c);
        }
        __syncthreads();
        for (uint32_t i = tid; i < 2 * S; i += kBucketThreads) {
            u64 *to = i < S ? a.load_data : a.load_parity;
            if (to) to[i < S ? i : i - S] += sh.list.srv[i];
        }
    }
    if (a.holding && b == 0 && tid == 0) hold_commit(a.hdr, a.packed != 0);       // nothing else of this launch reads these
    if (m == 0) return;
    if (tid <= a.tiles && tid < kMaxTiles) sh.pref[tid] = at;       // [tiles] = m as well (len is 0 there)
    if (tid == 0) sh.pref[a.tiles] = m;
    if (tid < a.tiles) sh.start[tid] = from;
    __syncthreads();
    // An ordinary bucket is one list; an oversized one comes in parts, one list after the other.
    const bool oversized = m > kBucketCap;
    uint32_t base = 0;                                              // items of the batch in earlier buckets
    bool have_base = oversized;
    PartWalk walk{0u, 0};
    if (oversized) {
        bucket_excl_scan(tid < a.tiles ? from - tid * a.tile : 0u, sh.wave, base);
        oversized_begin(a, sh, base);
    } else if (tid == 0) {
        sh.dense_used = 0;
    }
    uint32_t list = m;
    if (!oversized) {
        constexpr int P = kBucketCap / kBucketThreads;
        u64 it[P];
#pragma unroll
        for (int c = 0; c < P; ++c) {
            const uint32_t q = c * kBucketThreads + tid;
            if (q < m) it[c] = a.items[place_of(sh.pref, sh.start, a.tiles, q)];
        }
#pragma unroll
        for (int c = 0; c < P; ++c) {
            const uint32_t q = c * kBucketThreads + tid;
            if (q < m) sh.item[q] = it[c];
        }
        __syncthreads();
    }
    const RowArgs rows = a;
    const uint32_t shared = many ? a.lim.shared_stripe : 0u, packed = a.packed;
    for (;;) {
        if (oversized) list = oversized_part(args_again(), sh, m, base, walk);
        if (list) {
            sort_items(sh.item, sh.tmp, list, !oversized, sh.few);
            if (packed) {
                const BucketArgs b2 = args_again();
                for (uint32_t i = tid; i < list; i += kBucketThreads) sh.item[i] = resolved(b2, sh.item[i]);
                __syncthreads();
            }
            if (Rule<MODE>::combine) {
                const BucketArgs b2 = args_again();
                count_list(b2.geo, sh.item, list, sh.list.srv, b2.load_data, b2.load_parity);
            }
            apply_list<NC, MODE, PARITY, true, CUT>(rows, sh.item, list, heavy_run, shared, sh.list, (double *)sh.tmp);
            const uint32_t nh = uniform(sh.list.n_heavy);
            if (nh) {
                const BucketArgs b2 = args_again();
                if (!have_base) {
                    bucket_excl_scan(tid < b2.tiles ? from - tid * b2.tile : 0u, sh.wave, base);
                    have_base = true;
                }
                for (uint32_t h = 0; h < nh; ++h) {                 // the long runs' stripes, sorted as they are
                    const uint32_t at0 = uniform(sh.dense_used), hs = uniform(sh.list.heavy[h]);
                    const uint32_t start = hs & 0xFFFFu, count = (hs >> 16) - start;
                    for (uint32_t i = tid; i < count; i += kBucketThreads) b2.dense[base + at0 + i] = sh.item[start + i];
                    __syncthreads();                                // every wave has taken at0
                    if (tid == 0) list_heavy(b2, sh.dense_used, base, at0, count, true);
                    __syncthreads();
                }
            }
        }
        if (!oversized || walk.depth < 0) break;
    }
}

// ================================================================================================
// heavy stripes
// ================================================================================================

// (stripe, 16 columns) per workgroup: long_runs.h.
static_assert(kSplitSegment == kHeavyThreads / 8 * kHeavyT, "a segment is one round of a workgroup");

constexpr uint32_t kFoldParts = kHeavyThreads / kHeavyCols, kFoldLength = 16;       // of heavy_segment
static_assert(kFoldParts * kFoldLength * kSplitSegment >= kBucketMaxBatch && kHeavyThreads * kSplitSegment >= kBucketMaxBatch,
              "a run's segments are folded in one go, and waited for by a thread each");
struct HeavyShared {
    HeavyExchange ex[2];
    double part[2][kFoldParts][kHeavyCols], dec[kFoldParts];
    uint32_t pref[kMaxTiles + 1], start[kMaxTiles];
    uint32_t job, last;
};

// ---- runs that are cut into segments -------------------------------------------------------------
// With a batch on a handful of entries -- the smallest tables of a model, one very hot row -- a run has tens of thousands of
// updates, and D / 16 workgroups walking it at 3.5 us per 1024 are what everything waits for.  Such a stripe's runs are
// cut into segments of one round each.  A workgroup sums up its segment, publishes the sum, takes the sums of the segments
// before it for its starting state, computes its steps from the gradients it still has in registers, and leaves
// their sum; the last workgroup of the stripe (and 16 columns) to arrive applies the totals, entry by entry, segment by segment in order.
// The wait for earlier segments ends: jobs are handed out in ascending order by one counter, so whoever waits knows the
// earlier ones to be in the hands of workgroups that are already running, and those publish before they wait themselves.
// us a call, D = 128, one workgroup to a run and 16 columns / cut up: all of 2^14, 2^16, 2^18 updates on one row 92 / 35, 304 / 54,
// 1169 / 170; half of 2^18 706 / 222; 2^16 on 16 rows 104 / 65.

// What workgroups of one launch leave each other is written and read by relaxed atomics of device scope: they pass by the
// caches that the XCDs do not share.  published() waits until a wave's are done, so that a flag or a count written next is
// seen after them.  (Fences of device scope would write back and invalidate those caches as a whole, for every segment:
// 2^19 updates on 2^7 rows took 800 us with them.)
__device__ __forceinline__ double shared_load(const double *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void shared_store(double *p, double v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void published() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Folds the sums (ROWS = 1) or the sums and steps (2) of segments first .. first + count - 1, columns cg * 16 ..: kFoldParts
// threads per column take kFoldLength segments each and leave theirs in sh.part, with the decay in sh.dec.  The last
// segment's decay is last_dec, that of the others dec.  Ends with a barrier.
template <int MODE, int ROWS>
__device__ __forceinline__ void fold_segments(const BucketArgs &a, HeavyShared &sh, uint32_t first, uint32_t count, uint32_t cg,
                                              double dec, double last_dec)
{
    constexpr bool kMomentum = MODE == kMomentumSeq;
    const uint32_t c = threadIdx.x % kHeavyCols, part = threadIdx.x / kHeavyCols, col = cg * kHeavyCols + c, D = a.geo.D;
    constexpr uint32_t kAtOnce = 8;
    const uint32_t begin = part * kFoldLength, end = min(begin + kFoldLength, count);
    double s = -0.0, steps = 0.0, d = 1.0;
    for (uint32_t j0 = begin; j0 < end; j0 += kAtOnce) {
        double v[ROWS][kAtOnce];
#pragma unroll
        for (uint32_t i = 0; i < kAtOnce; ++i) {
            const bool in = j0 + i < end && col < D;
#pragma unroll
            for (int q = 0; q < ROWS; ++q)
                v[q][i] = in ? shared_load((q ? a.split.steps : a.split.sums) + (size_t)(first + j0 + i) * D + col) : 0.0;
        }
#pragma unroll
        for (uint32_t i = 0; i < kAtOnce; ++i) {
            if (j0 + i >= end) break;
            const double di = j0 + i + 1u == count ? last_dec : dec;
            s = kMomentum ? fma(di, s, v[0][i]) : s + v[0][i];
            if (kMomentum) d = decay(d * di, (double)a.geo.mu);
            if (ROWS == 2) steps += v[ROWS - 1][i];
        }
    }
    sh.part[0][part][c] = s;
    if (ROWS == 2) sh.part[1][part][c] = steps;
    if (c == 0) sh.dec[part] = d;
    __syncthreads();
}

// The last workgroup of a stripe applies what its segments have left: 16 columns, a thread each.
template <int MODE, bool PARITY>
__device__ __forceinline__ void finish_stripe(const BucketArgs &a, HeavyShared &sh, uint32_t h, uint32_t g, uint32_t cg)
{
    constexpr bool kMomentum = MODE == kMomentumSeq;
    const uint32_t D = a.geo.D, k = a.geo.k, tid = threadIdx.x, col = cg * kHeavyCols + tid;
    const RuleParams rp = rule_params(a.geo);
    const double dec = kMomentum ? decay_over(kSplitSegment, rp.mu) : 1.0;
    const bool mine = tid < kHeavyCols && col < D;
    double pe = 0, pa = 0;
    if (PARITY && mine) {
        pe = (double)a.PE[(size_t)g * D + col];
        pa = (double)a.PA[(size_t)g * D + col];
    }
    for (uint32_t j = 0; j < k; ++j) {
        const SplitRun run = a.split.run[h * k + j];
        if (run.updates == 0) continue;
        const uint32_t segs = (run.updates + kSplitSegment - 1) / kSplitSegment, x = g * k + j;
        const double last_dec = kMomentum ? decay_over(run.updates - (segs - 1) * kSplitSegment, rp.mu) : 1.0;
        fold_segments<MODE, 2>(a, sh, run.first, segs, cg, dec, last_dec);
        if (mine) {
            float *e = a.E + (size_t)x * D + col, *state0 = a.A + (size_t)x * D + col;
            const double e64 = (double)*e, a64 = (double)*state0;
            double state = Rule<MODE>::start(a64), acc = 0.0;
            for (uint32_t p = 0; p * kFoldLength < segs; ++p) {
                state = kMomentum ? fma(sh.dec[p], state, sh.part[0][p][tid]) : state + sh.part[0][p][tid];
                if (!Rule<MODE>::combine) acc += sh.part[1][p][tid];
            }
            Rule<MODE>::finish(state, acc, a64, rp);
            *e = (float)(e64 - acc);
            *state0 = (float)state;
            pe -= acc;
            pa += state - a64;
        }
        if (cg == 0 && tid == 0) {
            if (run.updates > kLongRun) {
                atomicAdd(&a.hdr->n_long, 1u);
                atomicAdd(&a.hdr->n_long_items, (u64)run.updates);
            }
            if (Rule<MODE>::combine) {
                atomicAdd(&a.load_data[a.geo.dS.mod(g + 1 + j)], 1ull);
                if (a.load_parity) atomicAdd(&a.load_parity[a.geo.dS.mod(g)], 1ull);
            }
        }
        __syncthreads();                                            // sh.part is free for the next entry
    }
    if (PARITY && mine) {
        a.PE[(size_t)g * D + col] = (float)pe;
        a.PA[(size_t)g * D + col] = (float)pa;
    }
}

// One segment, 16 columns.
template <int MODE, bool PARITY>
__device__ __forceinline__ void heavy_segment(const BucketArgs &a, HeavyShared &sh, uint32_t segment, uint32_t cg)
{
    constexpr bool kMomentum = MODE == kMomentumSeq;
    constexpr int T = kHeavyT;
    const uint32_t D = a.geo.D, k = a.geo.k, tid = threadIdx.x, lane = lane_id(), w = uniform(tid / kWave);
    const uint32_t col_lane = lane & 7u, sub = w * 8u + lane / 8u, ncg = (D + kHeavyCols - 1) / kHeavyCols;
    const RuleParams rp = rule_params(a.geo);
    const uint32_t r = a.split.segment_run[segment], h = r / k;
    const SplitRun run = a.split.run[r];
    const uint32_t nth = segment - run.first, L = run.updates, col = cg * kHeavyCols + 2u * col_lane;
    const bool live = col < D;                                      // D is a multiple of 4: both columns or none
    const uint32_t *tiles = a.split.tiles + (size_t)r * kSplitTileWords;
    for (uint32_t t = tid; t <= a.tiles; t += kHeavyThreads) {
        sh.pref[t] = tiles[t];
        if (t < a.tiles) sh.start[t] = tiles[kMaxTiles + 1 + t];
    }
    __syncthreads();
    // the eight lanes of a group look up two of its T updates each (past the run's end: the last one)
    const uint32_t off = nth * kSplitSegment + sub * T, q = off + 2u * col_lane;
    const u64 it0 = resolved(a, a.items[place_of(sh.pref, sh.start, a.tiles, min(q, L - 1u))]);
    const u64 it1 = resolved(a, a.items[place_of(sh.pref, sh.start, a.tiles, min(q + 1u, L - 1u))]);
    const uint32_t x = uniform(item_row(it0)), g = a.geo.dk.div(x);
    float2 gr[T];
    heavy_rows<T>(gr, a.grads, D, col, live, (uint32_t)it0, (uint32_t)it1, lane, off, L);
    const uint32_t cnt = off < L ? min((uint32_t)T, L - off) : 0u;
    D2 state = D2{0, 0};
    if (!Rule<MODE>::combine && live) state = widen2(*(const float2 *)(a.A + (size_t)x * D + col));
    double ed;
    const D2 ex = heavy_sums<MODE>(gr, cnt, rp, sh.ex[0], w, ed);
    __syncthreads();
    // ---- its sum, for the segments behind it (and for the run's end)
    if (w == 0 && lane < 8u && live) {
        D2 sum = D2{-0.0, -0.0};
        heavy_fold<MODE>(sum, sh.ex[0], w, ex, ed);
        double *to = a.split.sums + (size_t)segment * D + col;
        shared_store(to, sum.x);
        shared_store(to + 1, sum.y);
    }
    uint32_t *summed = a.split.summed + (size_t)run.first * ncg + cg;
    if (w == 0) {
        published();
        if (lane == 0) __hip_atomic_store(summed + (size_t)nth * ncg, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (!Rule<MODE>::combine) {
        // ---- the state it starts from
        if (tid < nth)                                              // nth < 512
            while (!__hip_atomic_load(summed + (size_t)tid * ncg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) __builtin_amdgcn_s_sleep(2);
        __syncthreads();
        const double dec = kMomentum ? decay_over(kSplitSegment, rp.mu) : 1.0;
        fold_segments<MODE, 1>(a, sh, run.first, nth, cg, dec, dec);
        for (uint32_t p = 0; p * kFoldLength < nth; ++p) {
            const double px = sh.part[0][p][2u * col_lane], py = sh.part[0][p][2u * col_lane + 1u], dp = kMomentum ? sh.dec[p] : 1.0;
            state.x = kMomentum ? fma(dp, state.x, px) : state.x + px;
            state.y = kMomentum ? fma(dp, state.y, py) : state.y + py;
        }
        // ---- its steps
        D2 mine = heavy_fold<MODE>(state, sh.ex[0], w, ex, ed), acc = D2{0, 0};
#pragma unroll
        for (int u = 0; u < T; ++u) {
            if ((uint32_t)u < cnt) item2<MODE>(mine, acc, gr[u], rp);
        }
        acc = heavy_total(acc, sh.ex[1], w);
        if (w == 0 && lane < 8u && live) {
            double *to = a.split.steps + (size_t)segment * D + col;
            shared_store(to, acc.x);
            shared_store(to + 1, acc.y);
        }
    }
    // ---- the last to arrive of the stripe's segments
    if (w == 0) {
        const uint32_t m = lane < k ? a.split.run[h * k + lane].updates : 0u;
        uint32_t all = (m + kSplitSegment - 1) / kSplitSegment;
#pragma unroll
        for (int by = 1; by < kWave; by <<= 1) all += __shfl_xor(all, by, kWave);
        published();
        if (lane == 0)
            sh.last = __hip_atomic_fetch_add(a.split.arrived + h * ncg + cg, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == all;
    }
    __syncthreads();
    if (uniform(sh.last)) finish_stripe<MODE, PARITY>(a, sh, h, g, cg);
}

template <int MODE, bool PARITY>
__global__ __launch_bounds__(kHeavyThreads) void heavy_stripes_kernel(BucketArgs a)
{
    constexpr int T = kHeavyT;
    __shared__ HeavyShared sh;
    if (a.hdr->batch_bad) return;
    plan_replay(a);
    const uint32_t nh = a.hdr->n_heavy, ns = a.hdr->n_segments, D = a.geo.D, k = a.geo.k, lane = lane_id();
    if (nh + ns == 0) return;
    const uint32_t w = uniform(threadIdx.x / kWave), col_lane = lane & 7u, sub = w * 8u + lane / 8u;
    const uint32_t ncg = (D + kHeavyCols - 1) / kHeavyCols;
    const RuleParams rp = rule_params(a.geo);
    // jobs are handed out as workgroups come free: their lengths differ by orders of magnitude
    auto next_job = [&]() {
        if (threadIdx.x == 0) sh.job = atomicAdd(&a.hdr->heavy_ticket, 1u);
        __syncthreads();
        return uniform(sh.job);
    };
    uint32_t job = next_job();
    for (; job < ns * ncg; job = next_job()) {                      // the segments first, in order: heavy_segment relies on it
        heavy_segment<MODE, PARITY>(a, sh, job / ncg, job % ncg);
        __syncthreads();
    }
    for (; job < (ns + nh) * ncg; job = next_job()) {
        const uint32_t h = job / ncg - ns, cg = job % ncg;
        const uint32_t start = a.heavy[2 * h], what = a.heavy[2 * h + 1], end = start + (what & ~kCounted);
        const u64 *items = a.dense;
        const uint32_t col = cg * kHeavyCols + 2u * col_lane;
        const bool live = col < D;                                  // D is a multiple of 4: both columns or none
        const uint32_t g = a.geo.dk.div(uniform(item_row(items[start])));
        D2 pe = D2{0, 0}, pa = D2{0, 0};
        if (PARITY && live) {
            pe = widen2(*(const float2 *)(a.PE + (size_t)g * D + col));
            pa = widen2(*(const float2 *)(a.PA + (size_t)g * D + col));
        }
        // Half of sh.ex for the next exchange.  It changes with every exchange and with nothing else: a half is written again
        // only behind the barrier of the exchange in between, which every wave passes after it has read the half.
        uint32_t buf = 0;
        for (uint32_t p = start; p < end;) {
            const uint32_t x = uniform(item_row(items[p]));
            uint32_t lo = p, hi = end;                              // items[lo] has row x; hi: the first that has not
            while (hi - lo > 1) {
                const uint32_t step = (hi - lo + kWave - 1) / kWave, probe = lo + (lane + 1u) * step;
                const uint32_t in = (uint32_t)__popcll(__ballot(probe < hi && item_row(items[min(probe, end - 1)]) == x));
                const uint32_t out = lo + (in + 1u) * step;
                lo += in * step;
                if (in < (uint32_t)kWave && out < hi) hi = out;
            }
            const uint32_t L = hi - p;
            float *erow = a.E + (size_t)x * D + col, *arow = a.A + (size_t)x * D + col;
            float2 e = float2{0, 0}, a0 = float2{0, 0};
            if (live) {
                e = *(const float2 *)erow;
                a0 = *(const float2 *)arow;
            }
            D2 state = start2<MODE>(widen2(a0)), acc = D2{0, 0};
            // The rows of a round are asked for while the round before is computed, its indices a round earlier.  The
            // eight lanes of a group fetch two of its T indices each.
            float2 gr[T], nx[T];
            uint32_t i0, i1;
            heavy_indices(items + p, L, sub * T + 2u * col_lane, i0, i1);
            heavy_rows<T>(nx, a.grads, D, col, live, i0, i1, lane, sub * T, L);
            heavy_indices(items + p, L, 64u * T + sub * T + 2u * col_lane, i0, i1);
            for (uint32_t r0 = 0; r0 < L; r0 += 64u * T) {
                const uint32_t off = r0 + sub * T;
                const uint32_t cnt = off < L ? min((uint32_t)T, L - off) : 0u;
#pragma unroll
                for (int u = 0; u < T; ++u) gr[u] = nx[u];
                if (r0 + 64u * T < L) {
                    heavy_rows<T>(nx, a.grads, D, col, live, i0, i1, lane, off + 64u * T, L);
                    heavy_indices(items + p, L, off + 128u * T + 2u * col_lane, i0, i1);
                }
                if (Rule<MODE>::combine) {                          // a sum: nothing to exchange before the run's end
#pragma unroll
                    for (int u = 0; u < T; ++u) {                   // zeros past the end of the run
                        acc.x += (double)gr[u].x;
                        acc.y += (double)gr[u].y;
                    }
                    continue;
                }
                double ed;
                const D2 ex = heavy_sums<MODE>(gr, cnt, rp, sh.ex[buf], w, ed);
                __syncthreads();
                D2 mine = heavy_fold<MODE>(state, sh.ex[buf], w, ex, ed);
#pragma unroll
                for (int u = 0; u < T; ++u) {
                    if ((uint32_t)u < cnt) item2<MODE>(mine, acc, gr[u], rp);
                }
                buf ^= 1u;
            }
            {                                                       // sum of the steps over groups, then over waves
                acc = heavy_total(acc, sh.ex[buf], w);
                buf ^= 1u;
                if (Rule<MODE>::combine) {
                    state = acc;
                    acc = D2{0, 0};
                }
            }
            const D2 e64 = widen2(e), a64 = widen2(a0);
            finish2<MODE>(state, acc, a64, rp);
            if (live && sub == 0) {
                *(float2 *)erow = narrow2(D2{e64.x - acc.x, e64.y - acc.y});
                *(float2 *)arow = narrow2(state);
            }
            pe.x -= acc.x;
            pe.y -= acc.y;
            pa.x += state.x - a64.x;
            pa.y += state.y - a64.y;
            if (cg == 0 && threadIdx.x == 0) {
                if (L > kLongRun) {                                 // reported by ecrm_batch_stats
                    atomicAdd(&a.hdr->n_long, 1u);
                    atomicAdd(&a.hdr->n_long_items, (u64)L);
                }
                if (Rule<MODE>::combine && !(what & kCounted)) {
                    atomicAdd(&a.load_data[a.geo.dS.mod(g + 1 + (x - g * k))], 1ull);
                    if (a.load_parity) atomicAdd(&a.load_parity[a.geo.dS.mod(g)], 1ull);
                }
            }
            p = hi;
        }
        if (PARITY && live && sub == 0) {
            *(float2 *)(a.PE + (size_t)g * D + col) = narrow2(pe);
            *(float2 *)(a.PA + (size_t)g * D + col) = narrow2(pa);
        }
        __syncthreads();                                            // what is in LDS is free for the next job
    }
}

// ================================================================================================
// host side
// ================================================================================================

template <int NC, int MODE, bool PARITY, bool CUT>
static void bucket_apply_as(const BucketArgs &a, bool heavy, int cus, hipStream_t st)
{
    static_assert(std::is_same_v<decltype(&bucket_apply_kernel<NC, MODE, PARITY, CUT>), void (*)(BucketArgs)>, "args_again reads one argument");
    const dim3 grid(a.buckets + kHotBuckets), block(kBucketThreads);
    const uint32_t most = a.n / kHeavyRunMin * ((a.geo.D + kHeavyCols - 1) / kHeavyCols);
    const dim3 hgrid(most < (uint32_t)cus ? most : (uint32_t)cus), hblock(kHeavyThreads);
    hipLaunchKernelGGL((bucket_apply_kernel<NC, MODE, PARITY, CUT>), grid, block, 0, st, a);
    if (heavy) hipLaunchKernelGGL((heavy_stripes_kernel<MODE, PARITY>), hgrid, hblock, 0, st, a);
}

template <int NC, int MODE>
static void bucket_apply_for(const BucketArgs &a, bool parity, bool heavy, int cus, hipStream_t st)
{
    const bool cut = lists_are_cut(a.geo.dk.div(a.geo.rows), a.buckets, a.n);
    if (parity) {
        if (cut) bucket_apply_as<NC, MODE, true, true>(a, heavy, cus, st);
        else bucket_apply_as<NC, MODE, true, false>(a, heavy, cus, st);
    } else {
        if (cut) bucket_apply_as<NC, MODE, false, true>(a, heavy, cus, st);
        else bucket_apply_as<NC, MODE, false, false>(a, heavy, cus, st);
    }
}

void launch_bucket_partition(const BucketScratch &bs, Header *hdr, const Geometry &g, const RecoveryView &rv,
                             const uint64_t *keys, uint32_t n, BatchSource src, bool clear_sticky, hipStream_t st)
{
    const BucketPlan p = bucket_plan(n);
    PartitionArgs a;
    a.keys = keys; a.items = bs.items; a.table = bs.table; a.tile_cnt = bs.tile_cnt; a.tile_state = bs.tile_state;
    a.hdr = hdr; a.n = n; a.tiles = p.tiles; a.buckets = p.buckets; a.rows = g.rows; a.D = g.D;
    a.count = (g.mode & 2u) ? 0u : 1u;               // the combined rules count per modified entry, later
    a.clear_sticky = clear_sticky ? 1u : 0u;
    a.packed = src == kWaitingUpdates ? 1u : 0u;
    a.dk = g.dk; a.dS = g.dS; a.rv = rv;
    const dim3 grid(p.tiles + 1u), block(kPartThreads);
    switch (p.ipt) {
        case 1: hipLaunchKernelGGL(bucket_partition_kernel<1>, grid, block, 0, st, a); break;
        case 2: hipLaunchKernelGGL(bucket_partition_kernel<2>, grid, block, 0, st, a); break;
        default: hipLaunchKernelGGL(bucket_partition_kernel<4>, grid, block, 0, st, a); break;
    }
}

void launch_bucket_apply(const BucketScratch &bs, Header *hdr, const Geometry &g, float *E, float *A, float *PE, float *PA,
                         unsigned long long *load_data, unsigned long long *load_parity, const uint64_t *keys,
                         uint32_t *rejected, const float *grads, uint32_t n, BatchSource src, bool holding, int cus, hipStream_t st)
{
    const BucketPlan p = bucket_plan(n);
    BucketArgs a;
    a.E = E; a.A = A; a.PE = PE; a.PA = PA; a.grads = grads; a.geo = g;
    a.keys = keys; a.items = bs.items; a.tmp = bs.tmp; a.dense = bs.dense; a.table = bs.table;
    a.tile_cnt = bs.tile_cnt; a.tile_state = bs.tile_state; a.heavy = bs.heavy; a.split = bs.split; a.hdr = hdr;
    a.load_data = load_data; a.load_parity = load_parity; a.rejected = rejected;
    a.n = n; a.tile = p.ipt * kPartThreads; a.tiles = p.tiles; a.buckets = p.buckets;
    a.packed = src == kWaitingUpdates ? 1u : 0u;
    a.holding = holding ? 1u : 0u;
    a.lim = bucket_limits(n, g.k, g.D);
    const bool heavy = n >= kHeavyRunMin;
    ECRM_DISPATCH(bucket_apply_for, a, PE != nullptr, heavy, cus, st);
}

}  // namespace ecrm
