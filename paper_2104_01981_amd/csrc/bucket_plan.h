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
constexpr uint32_t kBucketCap = 1024;        // items of a bucket that are sorted in LDS
constexpr uint32_t kBucketMaxServers = 64;   // per-tile load counts are kept for at most this many servers
constexpr uint32_t kBucketChunk = 8;         // sorted positions whose stripes a wave owns at a time
// A stripe with a run this long leaves its bucket and is split over the columns (heavy_stripes): one wave walks ~10 updates
// per us, the split takes ~5 us per 1024 but a workgroup for every 16 columns, so that there must not be many of them:
// at most 2048 runs of n / 2048.
constexpr uint32_t kHeavyRunMin = 128;
ECRM_HD uint32_t heavy_run(uint32_t n) { return n / 2048u > kHeavyRunMin ? n / 2048u : kHeavyRunMin; }
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
constexpr uint32_t kSmallSampled = kBucketCap * (kSample / 2) / 4;
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
