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

// Batches up to here go through buckets.  us a call with the sort and the chain tiers / with buckets, D = 128, k = 4, at 2^18 and at
// 2^19 updates: uniform on 4 n rows 306 / 233 and 537 / 438, on n / 8 rows 240 / 119 and 278 / 158; Zipf on n rows 448 / 195
// and 499 / 319; D = 512 on 4 n rows 672 / 691 (2 n rows) and 1584 / 1592; k = 10 on n / 16 rows 152 / 178 at 2^19.  Beyond, the sort's fixed cost is
// small; and a batch whose updates share few rows is slower in buckets from 300 000 updates on (2^19 on n / 32 rows 130 / 150).
constexpr uint32_t kBucketMaxBatch = 1u << 19;
// ... but for the larger half of them on the smallest tables, which the chain tiers spread better: 2^19 updates on 16, 32, 64,
// 128 rows take 179, 177, 175, 176 us there, in buckets 317, 449, 217, 154.
constexpr uint32_t kFewRows = 128, kFewRowsBatch = 1u << 18;
constexpr int kBucketThreads = 256;
constexpr int kPartThreads = 512;            // of the partition: 8 waves, 1, 2 or 4 updates per thread
constexpr uint32_t kMaxBuckets = 4096;
constexpr uint32_t kHotBuckets = 256;        // more, for the entries of hot stripes
// Of the workgroups of as many the first look after a hot stripe each, the others work off their columns.
constexpr uint32_t kHotMax = 64, kHotWorkers = kHotBuckets - kHotMax;
constexpr uint32_t kMaxTiles = 256;          // one thread per tile when a bucket is collected
// Items of a bucket that are sorted in LDS: what leaves room for the four workgroups of a compute unit that the registers
// allow.  2^19 updates on 2^13 rows (k = 10) take 395 us with 1024, 230 with 1536 and 289 with 2048; 2^16 Zipf 87, 88, 109.
constexpr uint32_t kBucketCap = 1536;
constexpr uint32_t kBucketMaxServers = 64;   // per-tile load counts are kept for at most this many servers
constexpr uint32_t kBucketChunk = 8;         // sorted positions whose stripes a wave owns at a time
// A stripe that does not end inside a window of 64 positions leaves its bucket for heavy_stripes, which splits it over the
// columns, if it has a run of heavy_run(n) updates: its workgroup would take 25 of them per us, where heavy_stripes takes 300
// but begins when the buckets are done.  With runs from 128 on heavy, n / 2048 in large batches: 8192 half Zipf 39.5, now 33.0;
// 65 536 half Zipf 89.4, 84.9; 300 007 Zipf combined 197, 182; 2^19 Zipf 324, 293.  Where heavy_stripes has hot stripes to
// work off anyway, behind the buckets, that shorter run (heavy_run_beside) is the better one, up to 128 floats: 26 features of
// 3 to 4096 rows and up, 131 072 updates 151 with heavy_run, 129 with heavy_run_beside, 262 144 with k = 10 338, 308; but
// 65 536 Zipf on 1024 rows of 512 floats 172, 254, where each entry of a stripe is worked on by 32 workgroups.  A
// heavy stripe takes ~6 us for every entry in each of its D / 16 workgroups, however short its run is, so that few of them
// are a gain and many a loss.  In a batch of many long stripes -- more than kManyHot hot ones in the sample: a small table --
// a stripe that no run dominates is shared by the waves of its workgroup instead, as long as it has fewer than
// shared_stripe(n, k) updates: that costs little of the chip's time but takes as long as its longest runs.  That limit lies
// where batches of nothing but such stripes break even: 256 updates in one of 2^14, 512 in one of 2^16, 1448 in one of 2^19
// (2^19 on 2^11 rows, D = 512: 1877 us when runs of 256 were always heavy, 557 shared); 16 updates to an entry (2^14 on 2520
// rows, k = 63: 281 and 63 us).  kManyHot lies between Zipf batches, of up to ~25 hot stripes (2^16 updates: 88 us with their
// long stripes shared, 80 with them heavy), and tables of a few hundred stripes, of 36 or more (2^16 on 1024 rows: 75 and 99).
constexpr uint32_t kManyHot = 32;
constexpr uint32_t kHeavyRunMin = 128, kHeavyStripeMin = 256, kHeavyEntryMin = 16;
ECRM_HD uint32_t heavy_run(uint32_t n) { return n / 640u > 2u * kHeavyRunMin ? n / 640u : 2u * kHeavyRunMin; }
ECRM_HD uint32_t heavy_run_beside(uint32_t n) { return n / 2048u > kHeavyRunMin ? n / 2048u : kHeavyRunMin; }
// of a stripe that makes its bucket too long for LDS
ECRM_HD uint32_t heavy_stripe(uint32_t k) { return kHeavyEntryMin * k > kHeavyStripeMin ? kHeavyEntryMin * k : kHeavyStripeMin; }
ECRM_HD uint32_t square_root(uint32_t v)     // rounded down; v below 2^24
{
    uint32_t root = 0;
    for (uint32_t bit = 1u << 11; bit; bit >>= 1)
        if ((root + bit) * (root + bit) <= v) root += bit;
    return root;
}
ECRM_HD uint32_t shared_stripe(uint32_t n, uint32_t k)
{
    const uint32_t root = square_root(4u * n);
    return root > heavy_stripe(k) ? root : heavy_stripe(k);
}
static_assert(kHeavyEntryMin * 64u <= kBucketCap && 4u * kBucketMaxBatch < kBucketCap * kBucketCap, "a stripe that is not heavy fits a list");
// A stripe of the sample with split_stripe(n, D) updates has its runs cut into segments, which go to as many workgroups as
// there are; a shorter one is walked by D / 16 workgroups, in rounds of kSplitSegment updates.  A round takes 3.5 us and a
// segment 17, so that a batch of nothing but such stripes breaks even where a stripe's rounds take as long as all the
// segments together.
constexpr uint32_t kSplitStripeMin = 8192, kSplitSegment = 1024;
ECRM_HD uint32_t split_stripe(uint32_t n, uint32_t D)
{
    const uint32_t even = n / 64u * ((D + 15u) / 16u);       // < 2^20 updates, 64 groups of columns: below 2^20
    return even > kSplitStripeMin ? even : kSplitStripeMin;
}
// segments of a batch of n updates: one per kSplitSegment, and a partly filled one for every run of such a stripe
ECRM_HD uint32_t split_segments(uint32_t n, uint32_t k)
{
    const uint32_t runs = n / kSplitStripeMin * k;
    return runs ? n / kSplitSegment + (runs < kHotBuckets ? runs : kHotBuckets) : 0u;
}
// Hot stripes are worked off beside the buckets, by workgroups that begin first, or by heavy_stripes behind them.  In place: one
// of up to this many updates, and of at most this many entries: each costs its workgroups a few more trips to memory than in
// heavy_stripes (2^16 updates on 2520 rows, k = 63: 594 us there, 782 in place).
constexpr uint32_t kInPlaceEntries = 16;
ECRM_HD uint32_t hot_in_place(uint32_t n) { return n / 16u > 2048u ? n / 16u : 2048u; }
struct BucketLimits { uint32_t shared_stripe, split_stripe, hot_in_place; };
ECRM_HD BucketLimits bucket_limits(uint32_t n, uint32_t k, uint32_t D)
{
    return BucketLimits{shared_stripe(n, k), split_stripe(n, D), hot_in_place(n)};
}
// updates from which on a stripe that the sample took for hot is one; candidates: how many the sample has
ECRM_HD uint32_t hot_least(const BucketLimits &l, uint32_t k, uint32_t candidates)
{
    const uint32_t half = l.shared_stripe / 2u;
    return candidates > kManyHot ? l.shared_stripe : half > heavy_stripe(k) ? half : heavy_stripe(k);
}
ECRM_HD bool in_place_size(const BucketLimits &l, uint32_t k, uint32_t m)
{
    return m <= l.hot_in_place && m < l.split_stripe && k <= kInPlaceEntries;
}
// ... and only where that is not what the launch then takes: a hot stripe in place takes ~70 updates per us and 7 us for each
// entry, in D / 16 workgroups of which 288 make progress at a time, heavy_stripes 350 updates per us and as much for an entry, of
// 256.  Measured in updates of the former: what a stripe's workgroups have to do here has to end with the buckets' work, ~15 us
// and the `rest` of the batch at 25 updates of 128 floats to one of these, or at least by as much later as it would keep
// heavy_stripes busy -- that is, longer than the longest stripe of the batch does, if that one is left to it for its size.
// Without this rule, and without any stripe in place / with it: 2^19 updates on 128 rows 321, 170 / 153; 2^18 on 256
// rows of 512 floats 554, 380 / 375; 2^18 Zipf on 1024 rows 304, 209 / 212; 8192 Zipf on 2040 rows, k = 10, 98, 72 / 73; 8192 half
// Zipf on 2048 rows 32, 48 / 32 (the constants are fitted to 290 such batches: 2 % above the better of the two).
struct HotStripe { uint32_t updates, entries; };
ECRM_HD bool in_place_time(const BucketLimits &l, uint32_t D, uint32_t hot, uint32_t rest, const HotStripe &longest, const HotStripe &s)
{
    const uint32_t jobs = hot * ((D + 15u) / 16u), wide = D > 128u ? D : 128u;
    const uint32_t here = (512u * s.entries + s.updates) * (jobs > 288u ? jobs : 288u) / 288u;
    const uint32_t behind = (512u * s.entries + s.updates / 5u) * (jobs > 256u ? jobs : 256u) / 256u;
    const bool is_left = longest.updates > l.hot_in_place || longest.updates >= l.split_stripe;
    const uint32_t left = is_left ? 512u * longest.entries + longest.updates / 5u : 0u;
    return here <= 1024u + rest * wide / 1792u + (behind > left ? behind - left : 0u);
}
static_assert((512u * kInPlaceEntries + kBucketMaxBatch / 16u) < (1u << 20) && kBucketMaxBatch <= (1u << 19),
              "times 64 stripes of 64 groups of columns, and updates times 1024 floats, in 32 bits");
struct BucketPlan { uint32_t ipt, tiles, buckets; };
// Tiles as small as kMaxTiles of them allow.  Buckets of 8 updates while that gives no more than the 1024 workgroups that
// are resident at once -- the fewer updates a wave walks one after the other the better (2048 uniform updates: 19.0 us with 16 to a bucket, 16.7 with 8, 17.4 with 4) --, of 64 from
// then on, of more when the largest number of buckets is reached.
ECRM_HD uint32_t bucket_count(uint32_t n)
{
    const uint32_t fine = n / 8u < 1024u ? n / 8u : 1024u, most = n / 64u > fine ? n / 64u : fine;
    return most < 1u ? 1u : most > kMaxBuckets ? kMaxBuckets : most;
}
// Buckets of a plan that are filled where `hot` stripes may be worked off beside them: as many as are resident at once beside these
// stripes' workgroups, which keep their places for 20 to 35 us.  The ones behind would begin when the first of the others end, and
// the call would wait for them.  The rest of the plan's buckets stay empty, which costs nothing.  Of larger plans many begin
// late anyway.  Not during a recovery, whose decoder takes places of its own (20 batches of 65 536 half Zipf 3383 us, with fewer
// buckets 3407).  us a call, all buckets filled / so: 65 536 Zipf on 2^16 rows 81.7 / 77.7, half Zipf on 2^18 90.4 / 85.9, combined
// 87.9 / 83.4; 12 000 Zipf on 2^14 44.5 / 42.3; 63 207 half Zipf, combined, on 27 920 rows of 64 floats 71.8 / 65.2; but 52 947 Zipf, momentum, k = 1,
// on 25 934 rows of 64 floats 64.9 / 69.5, 26 624 half Zipf on 2^20 54.3 / 54.7: 92 batches with rows of up to 128 floats 0.989 times as long,
// 25 with rows of up to 256 0.994, though fewer than 1024 of those are resident.  Where a batch's hot stripes are left to heavy_stripes all
// the same, which only one workgroup finds out, it makes no difference (18 batches, 1.000).
// Not with longer rows, nor where stripes have too many entries to be worked off beside the buckets: 29 batches with rows of more than
// 256 floats took 1.011 times as long (33 549 half Zipf on 3432 rows of 512 floats 111, 120).
ECRM_HD bool beside_pays(uint32_t k, uint32_t D) { return k <= kInPlaceEntries && D <= 256u; }
constexpr uint32_t kResidentBuckets = 1024;
ECRM_HD uint32_t buckets_beside(uint32_t buckets, uint32_t hot, uint32_t D)
{
    const uint32_t jobs = hot * ((D + 15u) / 16u), left = kResidentBuckets - (jobs < kHotWorkers ? jobs : kHotWorkers);
    return buckets <= kResidentBuckets && buckets > left ? left : buckets;
}
ECRM_HD BucketPlan bucket_plan(uint32_t n)
{
    BucketPlan p;
    p.ipt = n <= 1u * kPartThreads * kMaxTiles ? 1u : n <= 2u * kPartThreads * kMaxTiles ? 2u : 4u;
    p.tiles = (n + p.ipt * kPartThreads - 1) / (p.ipt * kPartThreads);
    p.buckets = bucket_count(n);
    return p;
}
static_assert(kBucketMaxBatch <= 4u * kPartThreads * kMaxTiles, "the plan's largest tile covers the largest batch");

// A bucket's list of fewer than kSplitStripes stripes is cut at entries (apply_split in lists.h), by a kernel of its own where the table
// has fewer stripes than that for each bucket.  On larger ones such a list is an exception, and what the kernel takes for it --
// scalar registers, instructions -- costs all other lists: 81 batches on such tables 0.991 times as long without.
// Nor where the batch has kSplitUpdates updates for each stripe of the table: then few lists are short enough.  us a call, cut / not: 2^19
// uniform updates on 16 384 rows (128 to a stripe) 126.4 / 124.1, on 22 000 (95) 135.4 / 132.8, 2^18 on 11 200 (94) 86.0 / 84.1, 2^17 on
// 14 000, k = 10 (94) 62.9 / 61.7; but 8192 on 1000, k = 10 (82) 26.1 / 27.0, 466 158 on 407 862, k = 63, combined (72) 288 / 298, 2^17 on
// 20 000, k = 10 (66) 68.0 / 69.4, 2^18 on 16 384 (64) 101.1 / 104.0.
constexpr uint32_t kSplitStripes = 16, kSplitUpdates = 88;
ECRM_HD bool lists_are_cut(uint32_t stripes, uint32_t buckets, uint32_t n) { return stripes < kSplitStripes * buckets && n / kSplitUpdates < stripes; }

// Batches of up to kDirectBatch updates take one launch, in which every workgroup reads all of the keys (direct.hip).  us a call
// through the three launches of the buckets / so, D = 128, k = 4: 512 uniform updates 15.3 / 9.5, 2048 16.2 / 10.4, 3072
// 19.2 / 14.0; Zipf, 2048 on 2^16 rows 24.4 / 18.1, on 256 rows 27.7 / 17.7; on one row, on four, on 64: 2048 40.8 / 31.1, 51.4 / 40.1,
// 21.9 / 16.0, 3072 52.9 / 42.6, 63.8 / 51.8, 25.4 / 21.6; D = 1024, 2048 44.2 / 33.4, 54.8 / 46.8, 81.5 / 73.2, 3072
// 55.5 / 45.1, 66.9 / 58.7, 89.6 / 86.9; 650 batches of 1 to 3072 updates, rows of 4 to 1024 floats, k of 1 to 63 and all rules take
// 0.70 times as long, the slowest one 0.99.  4096 would gain as well (20.6 / 16.2), but not 4096 on four rows (51 / 145).
constexpr uint32_t kDirectBatch = 3072, kDirectLong = 192, kDirectWorkers = 128;
ECRM_HD uint32_t direct_buckets(uint32_t n) { return n / 8u > 1u ? n / 8u : 1u; }
ECRM_HD uint32_t direct_groups(uint32_t D) { return (D + 7u) / 8u; }
ECRM_HD uint32_t direct_workers(uint32_t jobs, uint32_t empty) { return jobs <= kDirectWorkers ? kDirectWorkers : kDirectWorkers + empty; }
// A bucket of kDirectLong updates or more may have a stripe that kDirectWorkers workgroups take instead of its own, eight columns each
// (and those whose bucket is empty, if that makes more jobs than these take at once).  By columns a run of kDirectRun updates or more
// is a trip to memory and an exchange, whatever its length, and the shorter runs go all at once; its own workgroup takes ~22 updates
// per us, so that it is the better one for a few hundred updates of several entries alike.  Both in eighths of a us, fitted to
// batches of 3000 updates on equally many stripes; D > 128 costs its own workgroup so much more.  How many other such stripes there
// are no workgroup but those of the columns knows: in a table of few stripes as many as there is room for, otherwise as a power law has
// them.  us a call through the buckets' launches / every long stripe by columns, 128 workgroups / so: 3000 on 56 rows, k = 4, D = 128
// 25.9 / 44.0 / 22.6, D = 1024 97 / 343 / 92; on 100, k = 10, D = 256 48.6 / 143.5 / 45.1; on 882, k = 63, D = 256 48.6 / 98.1 / 42.3; on
// ten, k = 1, D = 1024 61.8 / 123.0 / 42.7; but 2048 Zipf on 1020 rows, k = 10, 65.8 / 45.6 / 53.8: there it finds too few.
constexpr uint32_t kDirectRun = 32;
// a bucket's list: updates, entries, entries with kDirectRun updates or more, the other entries' updates; a run that is a third of it?
struct DirectList { uint32_t updates, entries, longer, others; bool third; };
ECRM_HD bool direct_by_columns(const DirectList &s, uint32_t n, uint32_t stripes, uint32_t D, bool combine)
{
    const uint32_t like = stripes < n / 128u ? n / s.updates : s.updates / kDirectLong;
    const uint32_t jobs = like * direct_groups(D), workers = kDirectWorkers + direct_buckets(n), turns = (jobs + workers - 1u) / workers;
    const uint32_t here = 16u + s.updates * 4u / 11u + 3u * s.entries + (s.third && s.entries > 1u ? 24u : 0u);
    const uint32_t run = (jobs <= kDirectWorkers ? 29u : turns == 1u ? 40u : 52u) >> (combine ? 1 : 0);
    const uint32_t rest = s.entries > s.longer ? 24u + 4u * s.others / (s.entries - s.longer) : 0u;
    return 8u + turns * (8u + s.entries + run * s.longer + rest) <= (D > 170u ? here * 3u * D / 512u : here);
}
// updates from which on a list's stripes go by columns whatever its runs are, so that nobody has to count them (0.5 us)
ECRM_HD uint32_t direct_sure(uint32_t n, uint32_t stripes, uint32_t k, uint32_t D, bool combine)
{
    uint32_t lo = kDirectLong - 1u, hi = n + 1u;
    while (hi > lo + 1u) {
        const uint32_t m = (lo + hi) / 2u, longer = k < m / kDirectRun ? k : m / kDirectRun;
        if (direct_by_columns(DirectList{m, k, longer, m, false}, n, stripes, D, combine)) hi = m; else lo = m;
    }
    return hi;
}

// Bijective mix of a stripe number: its low bits split a bucket further, and number the slots of tables in LDS.
ECRM_HD uint32_t scramble32(uint32_t g)
{
    g ^= g >> 16;
    g *= 0x9E3779B1u;
    g ^= g >> 15;
    g *= 0xD1B54A33u;
    return g ^ (g >> 16);
}
// Its high part selects the bucket.  Multiples of the golden ratio spread any range of numbers evenly, so that buckets of a
// table whose every stripe is touched get equally many; at random, as by the mix above, 4096 stripes in 1024 buckets are up
// to 13 to a bucket, and the call waits for that one (65 536 updates on 2^14 rows 47.1 us, now 43.2; 300 007 on 100 000 136, now 130).  The multiples start over somewhere else every 4096 stripes, so that
// a batch of one stripe out of a few thousand is spread as by the mix: a stride that meets a Fibonacci number would keep
// the multiples themselves close together.
ECRM_HD uint32_t mix32(uint32_t g) { return (g & 4095u) * 0x9E3779B1u + scramble32(g >> 12); }
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
    return lo + (uint32_t)(((uint64_t)scramble32(i) * (hi - lo)) >> 32);
}
// What `hits` of the sample, on `seen` different entries, say of a stripe: its updates; its entries, all that were seen if
// most hits repeat an entry, and by the number of repeats (as of birthdays) otherwise.
ECRM_HD uint32_t sampled_updates(uint32_t hits, uint32_t n) { return (uint32_t)(((uint64_t)hits * n) >> sample_bits(n)); }
ECRM_HD uint32_t sampled_entries(uint32_t hits, uint32_t seen, uint32_t k)
{
    const uint32_t guess = hits * hits / (2u * (hits - seen) + 1u), entries = hits >= 3u * seen ? seen : guess > seen ? guess : seen;
    return entries < k ? entries : k;
}
// hits from which on a stripe counts as hot
ECRM_HD uint32_t hot_hits(uint32_t n)
{
    const uint32_t hits = ((kHotRun << sample_bits(n)) + n - 1u) / n;
    return hits > 4u ? hits : 4u;
}

}  // namespace ecrm
