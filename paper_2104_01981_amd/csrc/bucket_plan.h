// How a batch of up to kBucketMaxBatch updates is cut into tiles and buckets, and which of its keys the partition looks at
// to find hot stripes (buckets.hip).  Plain arithmetic that the kernels and the host share; it compiles without HIP, so that
// a test can ask the very same functions.
#pragma once

#include <stdint.h>

#ifdef __HIP__
#define ECRM_HD __host__ __device__ __forceinline__
#else
#define ECRM_HD inline
#endif

namespace ecrm {

constexpr uint32_t kBucketMaxBatch = 1u << 19;
constexpr int kBucketThreads = 256;
constexpr int kPartThreads = 512;            // of the partition: 8 waves, 1, 2 or 4 updates per thread
constexpr uint32_t kMaxBuckets = 4096;
constexpr uint32_t kHotBuckets = 256;        // more, for the entries of hot stripes
constexpr uint32_t kMaxTiles = 256;          // one thread per tile when a bucket is collected
// Items of a bucket that are sorted in LDS: what leaves room for the four workgroups of a compute unit that the registers
// allow.  2^19 updates on 2^13 rows (k = 10) take 395 us with 1024, 230 with 1536 and 289 with 2048; 2^16 Zipf 87, 88, 109.
constexpr uint32_t kBucketCap = 1536;
constexpr uint32_t kBucketMaxServers = 64;   // per-tile load counts are kept for at most this many servers
constexpr uint32_t kBucketChunk = 8;         // sorted positions whose stripes a wave owns at a time
// A stripe that does not end inside a window of 64 positions leaves its bucket for heavy_stripes, which splits it over the
// columns, if one run of heavy_run(n) updates or more makes up more than half of it: the wave that owns it would need a
// quarter of a microsecond for each.  One whose updates are spread over its entries is shared by the waves of its
// workgroup, as long as it has fewer than shared_stripe(n, k) updates: sharing costs little of the chip's time but takes
// as long as its longest runs, a heavy stripe takes ~6 us for every entry in each of its D / 16 workgroups however short
// its run is, so that few of them are a gain and many a loss.  The limits lie where batches of nothing but such
// stripes break even: 256 updates in one of 2^14, 512 in one of 2^16, 1448 in one of 2^19 (2^19 on 2^11 rows, D = 512: 1877 us
// when runs of 256 were always heavy, 557 shared); 16 updates to an entry (2^14 on 2520 rows, k = 63: 281 and 63 us).
constexpr uint32_t kHeavyRunMin = 128, kHeavyStripeMin = 256, kHeavyEntryMin = 16;
ECRM_HD uint32_t heavy_run(uint32_t n) { return n / 2048u > kHeavyRunMin ? n / 2048u : kHeavyRunMin; }
// of a stripe that makes its bucket too long for LDS
ECRM_HD uint32_t heavy_stripe(uint32_t k) { return kHeavyEntryMin * k > kHeavyStripeMin ? kHeavyEntryMin * k : kHeavyStripeMin; }
ECRM_HD uint32_t shared_stripe(uint32_t n, uint32_t k)
{
    uint32_t root = 0;                       // of 4 n, rounded down
    for (uint32_t bit = 1u << 11; bit; bit >>= 1)
        if ((root + bit) * (root + bit) <= 4u * n) root += bit;
    return root > heavy_stripe(k) ? root : heavy_stripe(k);
}
static_assert(kHeavyEntryMin * 64u <= kBucketCap, "a stripe that is not heavy fits a list");
struct BucketPlan { uint32_t ipt, tiles, buckets; };
// Tiles as small as kMaxTiles of them allow.  Buckets of 16 updates while that gives no more than the 1024 workgroups that
// are resident at once -- the fewer updates a wave walks one after the other the better --, of 64 from then on, of more
// when the largest number of buckets is reached.
ECRM_HD BucketPlan bucket_plan(uint32_t n)
{
    BucketPlan p;
    p.ipt = n <= 1u * kPartThreads * kMaxTiles ? 1u : n <= 2u * kPartThreads * kMaxTiles ? 2u : 4u;
    p.tiles = (n + p.ipt * kPartThreads - 1) / (p.ipt * kPartThreads);
    const uint32_t fine = n / 16u < 1024u ? n / 16u : 1024u, most = n / 64u > fine ? n / 64u : fine;
    p.buckets = most < 1u ? 1u : most > kMaxBuckets ? kMaxBuckets : most;
    return p;
}
static_assert(kBucketMaxBatch <= 4u * kPartThreads * kMaxTiles, "the plan's largest tile covers the largest batch");

// Bijective mix of a stripe number: the high part selects the bucket, the low bits split a bucket further.
ECRM_HD uint32_t mix32(uint32_t g)
{
    g ^= g >> 16;
    g *= 0x9E3779B1u;
    g ^= g >> 15;
    g *= 0xD1B54A33u;
    return g ^ (g >> 16);
}
ECRM_HD uint32_t bucket_of(uint32_t g, uint32_t buckets) { return (uint32_t)(((uint64_t)mix32(g) * buckets) >> 32); }

// The sample in which stripes with about kHotRun updates or more are looked for: one key out of each of 2^sample_bits(n)
// equal segments of the batch.  A batch of up to kSmallSampled updates gets along with half the sample: what that is
// likely to miss is shorter than what a bucket holds.
constexpr uint32_t kHotRun = 256;
constexpr uint32_t kSample = 1024;
constexpr uint32_t kSmallSampled = 1u << 17;
ECRM_HD uint32_t sample_bits(uint32_t n) { return n <= kSmallSampled ? 9u : 10u; }
static_assert(kSample == 1u << 10, "sample_bits");
// Which key of its segment is looked at varies from segment to segment, the same way in every call: at a fixed distance the
// sample falls in with any period of the batch (keys of several tables taking turns: of a batch whose odd positions
// were the skewed ones it saw the even ones only, and missed a stripe of 12 404 of 2^19 updates).
ECRM_HD uint32_t sample_position(uint32_t i, uint32_t n)
{
    const uint32_t bits = sample_bits(n);
    const uint32_t lo = (uint32_t)(((uint64_t)i * n) >> bits), hi = (uint32_t)(((uint64_t)(i + 1u) * n) >> bits);
    return lo + (uint32_t)(((uint64_t)mix32(i) * (hi - lo)) >> 32);
}
// hits from which on a stripe counts as hot
ECRM_HD uint32_t hot_hits(uint32_t n)
{
    const uint32_t hits = ((kHotRun << sample_bits(n)) + n - 1u) / n;
    return hits > 4u ? hits : 4u;
}

}  // namespace ecrm
