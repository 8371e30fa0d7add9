// Training while a server is being recovered (Sec. 3.4 "Training during recovery"): updates that
// touch the chunk of stripes under reconstruction, and updates to lost entries that are not rebuilt
// yet, are not applied but appended -- in arrival order -- to a buffer of (key, gradient row) pairs,
// and replayed when their chunk is released.  The buffer is a pool of gradient rows addressed by
// slot plus a list of (key, slot) entries: a row is copied once, when its update is first held back;
// a replay only rewrites the list (what must go on waiting keeps its row) and releases the slots of
// what it applies.  This file holds the order-preserving append and replay bookkeeping (flag, block
// counts, scan, scatter).
#include "ecrm_internal.h"

namespace ecrm {

constexpr int kHoldThreads = 256;
constexpr int kHoldIpt = 8;                        // items per thread
static_assert(kHoldTile == kHoldThreads * kHoldIpt, "a tile is what a workgroup looks at");

typedef __amdgpu_buffer_rsrc_t rsrc_t;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t block_sum(uint32_t v, uint32_t *s_w)
{
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) v += __shfl_xor(v, d, kWave);
    if (lane_id() == 0) s_w[threadIdx.x / kWave] = v;
    __syncthreads();
    uint32_t t = 0;
    for (int w = 0; w < kHoldThreads / kWave; ++w) t += s_w[w];
    __syncthreads();
    return t;
}

// Is item i of the batch held back?  A caller's key is checked for range here as well (the first sort
// pass rejects the batch for it); a waiting update's key sits in the low half of its list entry.
__device__ __forceinline__ bool item_held(const uint64_t *keys, uint32_t i, uint32_t rows, const Divider &dk, const Divider &dS,
                                          const RecoveryView &rv, bool packed)
{
    const uint64_t x = keys[i];
    if (!packed && x >= (uint64_t)rows) return false;
    return held_back(rv, (uint32_t)x, dk, dS);
}

// pass 1: how many items of each tile are held back
__global__ __launch_bounds__(kHoldThreads) void hold_count_kernel(const uint64_t *keys, uint32_t n, const uint32_t *n_dev,
                                                                  uint32_t rows, Divider dk, Divider dS, RecoveryView rv,
                                                                  uint32_t packed, uint32_t *tile_count)
{
    __shared__ uint32_t s_w[kHoldThreads / kWave];
    if (n_dev) n = min(n, *n_dev);
    uint32_t c = 0;
    const uint32_t base = blockIdx.x * kHoldTile;
#pragma unroll
    for (int r = 0; r < kHoldIpt; ++r) {
        const uint32_t i = base + r * kHoldThreads + threadIdx.x;
        if (i < n && item_held(keys, i, rows, dk, dS, rv, packed != 0)) ++c;
    }
    const uint32_t t = block_sum(c, s_w);
    if (threadIdx.x == 0) tile_count[blockIdx.x] = t;
}

// pass 2 (one block): exclusive scan of the tile counts; totals and the capacity check
__global__ __launch_bounds__(1024) void hold_scan_kernel(uint32_t *tile_count, uint32_t ntiles, Header *hdr, uint32_t n,
                                                         const uint32_t *n_dev, uint32_t packed, uint32_t buf_cap)
{
    __shared__ uint32_t s_w[16];
    __shared__ uint32_t s_carry;
    if (n_dev) n = min(n, *n_dev);
    if (threadIdx.x == 0) s_carry = 0;
    __syncthreads();
    for (uint32_t b0 = 0; b0 < ntiles; b0 += 1024) {
        const uint32_t i = b0 + threadIdx.x;
        const uint32_t v = i < ntiles ? tile_count[i] : 0;
        uint32_t incl = v;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const uint32_t t = __shfl_up(incl, d, kWave);
            if (lane_id() >= (uint32_t)d) incl += t;
        }
        if (lane_id() == kWave - 1) s_w[threadIdx.x / kWave] = incl;
        __syncthreads();
        uint32_t off = s_carry, tot = 0;
        for (uint32_t w = 0; w < 16; ++w) {
            if (w < threadIdx.x / kWave) off += s_w[w];
            tot += s_w[w];
        }
        if (i < ntiles) tile_count[i] = off + incl - v;
        __syncthreads();
        if (threadIdx.x == 0) s_carry += tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const uint32_t held = s_carry;
        hdr->n_held = held;
        hdr->n_valid = n - held;
        // no room: the batch is rejected as a whole (a replay only ever shrinks the list)
        if (!packed && (unsigned long long)hdr->buf_count + held > buf_cap) {
            hdr->batch_bad = 1;
            hdr->err_sticky |= 2u;
        }
    }
}

// pass 3, a caller's batch: every held-back item gets a slot of the row pool -- released slots first,
// last released first, then slots never used -- its gradient row is copied there, and (key, slot) is
// appended to the list in arrival order.
// pass 3, a replay of the list: what must go on waiting is appended to the other list as it is (its row
// stays where it is); the slots of what is applied now are released, in list order.
__global__ __launch_bounds__(kHoldThreads) void hold_scatter_kernel(const uint64_t *keys, const float *grads, uint32_t n,
                                                                    const uint32_t *n_dev, uint32_t rows, uint32_t D,
                                                                    Divider dk, Divider dS, RecoveryView rv, uint32_t packed,
                                                                    const uint32_t *tile_offset, Header *hdr,
                                                                    unsigned long long *list_out, float *pool,
                                                                    uint32_t *free_list)
{
    __shared__ uint32_t s_src[kHoldTile];          // item index of the tile's held-back items, in order
    __shared__ uint32_t s_wcount[kHoldThreads / kWave][kHoldIpt];
    if (hdr->batch_bad) return;
    if (n_dev) n = min(n, *n_dev);
    const uint32_t base = blockIdx.x * kHoldTile;
    if (base >= n) return;
    const uint32_t lane = lane_id(), wave = threadIdx.x / kWave;
    // tile order is (r, thread): ballots give each item its rank among the held-back ones
    bool held[kHoldIpt];
    uint32_t below[kHoldIpt];
#pragma unroll
    for (int r = 0; r < kHoldIpt; ++r) {
        const uint32_t i = base + r * kHoldThreads + threadIdx.x;
        held[r] = i < n && item_held(keys, i, rows, dk, dS, rv, packed != 0);
        const unsigned long long m = __ballot(held[r]);
        below[r] = (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
        if (lane == 0) s_wcount[wave][r] = (uint32_t)__popcll(m);
    }
    __syncthreads();
    const uint32_t held_before_tile = tile_offset[blockIdx.x];
    const uint32_t free0 = hdr->free_count, bump0 = hdr->bump;
    uint32_t total = 0;
#pragma unroll
    for (int r = 0; r < kHoldIpt; ++r) {
        uint32_t before = total;                   // held-back items of earlier (r, wave) groups
        for (uint32_t w = 0; w < kHoldThreads / kWave; ++w) {
            if (w < wave) before += s_wcount[w][r];
            total += s_wcount[w][r];
        }
        const uint32_t pos = r * kHoldThreads + threadIdx.x;          // place in the tile
        const uint32_t i = base + pos;
        const uint32_t hrank = before + below[r];                     // held-back items of the tile before this one
        if (held[r]) s_src[hrank] = i;
        if (packed && i < n) {
            if (held[r]) list_out[held_before_tile + hrank] = keys[i];                    // goes on waiting, row in place
            else free_list[free0 + (base - held_before_tile) + (pos - hrank)] = (uint32_t)(keys[i] >> 32);   // slot released
        }
    }
    if (packed) return;
    __syncthreads();
    const uint32_t first = held_before_tile;       // rank of the tile's first held-back item in this batch
    const uint32_t list0 = hdr->buf_count;
    // row copies: U rows in flight per wave (one at a time the copy ran at 2 TB/s)
    constexpr uint32_t U = 8, W = kHoldThreads / kWave;
    for (uint32_t t0 = wave * U; t0 < total; t0 += W * U) {
        uint32_t slot[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t rk = first + min(t0 + u, total - 1);       // rank among the batch's held-back items
            slot[u] = rk < free0 ? free_list[free0 - 1u - rk] : bump0 + (rk - free0);
            slot[u] = (uint32_t)__builtin_amdgcn_readfirstlane((int)slot[u]);
        }
        for (uint32_t off = lane * 16u; off < D * 4u; off += kWave * 16u) {
            u32x4 v[U];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                const uint32_t i = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_src[min(t0 + u, total - 1)]);
                const rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(grads + (size_t)i * D), 0, (int)(D * 4u), 0x00020000);
                v[u] = __builtin_amdgcn_raw_buffer_load_b128(src, (int)off, 0, 2);
            }
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                if (t0 + u < total) {
                    const rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(pool + (size_t)slot[u] * D, 0, (int)(D * 4u), 0x00020000);
                    __builtin_amdgcn_raw_buffer_store_b128(v[u], out, (int)off, 0, 0);
                }
            }
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u)
            if (lane == u && t0 + u < total)
                list_out[(size_t)list0 + first + t0 + u] = keys[s_src[t0 + u]] | ((unsigned long long)slot[u] << 32);
    }
}

__global__ void hold_commit_kernel(Header *hdr, uint32_t packed)
{
    if (threadIdx.x != 0 || hdr->batch_bad) return;
    hold_commit(hdr, packed != 0);
}

// The three passes in one launch, for a batch that the partition (buckets.hip) has been over: it has counted what is held
// back in each of its tiles, at most kMaxTiles of them, so that every workgroup adds up those before its own.  A workgroup
// takes one of the partition's tiles, and its rows are a flat copy, 16 bytes a lane.  20 batches of 65 536 and ten replays,
// a fifth of each held back: four launches of 46 us together in tiles of 2048 -- 32 workgroups --, now one of 8 us, 4 for a replay.
// The header is brought up to date by bucket_apply: here every workgroup reads it.
struct HoldArgs {
    const uint64_t *keys;
    const float *grads;
    const uint32_t *tile_state;
    uint32_t n, tiles, rows, packed, cap;
    Geometry geo;
    Divider d4;
    RecoveryView rv;
    Header *hdr;
    unsigned long long *list_out;
    float *pool;
    uint32_t *free_list;
};

template <int IPT>
__global__ __launch_bounds__(kPartThreads) void hold_tiles_kernel(HoldArgs a)
{
    constexpr uint32_t kTile = kPartThreads * IPT, kWaves = kPartThreads / kWave;
    static_assert(kMaxTiles <= kPartThreads, "a thread per tile");
    __shared__ uint2 s_row[kTile];                 // the tile's held-back items, in order: item, slot
    __shared__ uint32_t s_before[kWaves], s_all[kWaves], s_cnt[kWaves][IPT];
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
    const uint32_t n = a.packed ? min(a.n, a.hdr->n_batch) : a.n;
    const uint32_t free0 = a.hdr->free_count, bump0 = a.hdr->bump, list0 = a.packed ? 0u : a.hdr->buf_count;
    const uint32_t state = tid < a.tiles ? a.tile_state[tid] : 0u;
    uint32_t all = state >> 1, before = tid < blockIdx.x ? all : 0u;
    const bool bad = __syncthreads_or(state & 1u);
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) {
        all += __shfl_xor(all, d, kWave);
        before += __shfl_xor(before, d, kWave);
    }
    if (lane == 0) {
        s_all[wave] = all;
        s_before[wave] = before;
    }
    // the tile's items in the partition's order -- (wave, r, lane) --, ranked among the held-back ones by ballots
    const uint32_t tile0 = blockIdx.x * kTile;
    uint64_t key[IPT];
    uint32_t below[IPT], held = 0;
#pragma unroll
    for (int r = 0; r < IPT; ++r) {
        const uint32_t i = tile0 + wave * (kWave * IPT) + r * kWave + lane;
        key[r] = i < n ? a.keys[i] : 0ull;
        const bool h = i < n && (a.packed || key[r] < (uint64_t)a.rows) && held_back(a.rv, (uint32_t)key[r], a.geo.dk, a.geo.dS);
        const unsigned long long m = __ballot(h);
        held |= h ? 1u << r : 0u;
        below[r] = (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
        if (lane == 0) s_cnt[wave][r] = (uint32_t)__popcll(m);
    }
    __syncthreads();
    all = before = 0;
#pragma unroll
    for (uint32_t w = 0; w < kWaves; ++w) {
        all += s_all[w];
        before += s_before[w];
    }
    // no room: the batch is rejected as a whole (a replay only ever shrinks the list)
    const bool full = !a.packed && (uint64_t)list0 + all > a.cap;
    if (blockIdx.x == 0 && tid == 0) {
        a.hdr->n_held = all;
        a.hdr->n_valid = n - all;
        if (bad || full) {
            a.hdr->batch_bad = 1;
            a.hdr->err_sticky |= (bad ? 1u : 0u) | (full ? 2u : 0u);
        }
    }
    if (bad || full) return;                       // the same in every workgroup
    uint32_t own = 0, at = 0;
#pragma unroll
    for (uint32_t w = 0; w < kWaves; ++w) {
#pragma unroll
        for (int r = 0; r < IPT; ++r) {
            if (w < wave) at += s_cnt[w][r];
            own += s_cnt[w][r];
        }
    }
#pragma unroll
    for (int r = 0; r < IPT; ++r) {
        const uint32_t pos = wave * (kWave * IPT) + r * kWave + lane, i = tile0 + pos, rank = at + below[r];
        at += s_cnt[wave][r];
        if (i >= n) continue;
        if (a.packed) {
            if ((held >> r) & 1u) a.list_out[before + rank] = key[r];                       // goes on waiting, row in place
            else a.free_list[free0 + (tile0 - before) + (pos - rank)] = (uint32_t)(key[r] >> 32);   // slot released
        } else if ((held >> r) & 1u) {             // a released slot, the last first, or one never used
            const uint32_t nth = before + rank;
            const uint32_t slot = nth < free0 ? a.free_list[free0 - 1u - nth] : bump0 + (nth - free0);
            a.list_out[(size_t)list0 + nth] = key[r] | ((unsigned long long)slot << 32);
            s_row[rank] = uint2{i, slot};
        }
    }
    if (a.packed) return;
    __syncthreads();
    constexpr uint32_t U = 4;
    const uint32_t D = a.geo.D, total = own * (D / 4u);
    for (uint32_t u0 = 0; u0 < total; u0 += U * kPartThreads) {
        float4 v[U];
        size_t to[U];
#pragma unroll
        for (uint32_t q = 0; q < U; ++q) {
            const uint32_t u = min(u0 + q * kPartThreads + tid, total - 1u), r = a.d4.div(u), c = (u - r * a.d4.d) * 4u;
            const uint2 what = s_row[r];
            v[q] = load4(a.grads + (size_t)what.x * D + c);
            to[q] = (size_t)what.y * D + c;
        }
#pragma unroll
        for (uint32_t q = 0; q < U; ++q)
            if (u0 + q * kPartThreads + tid < total) *(float4 *)(a.pool + to[q]) = v[q];
    }
}

void launch_hold_back(Header *hdr, uint32_t *tile_count, const Geometry &g, const RecoveryView &rv, const uint64_t *keys,
                      const float *grads, uint32_t n, BatchSource src, const HoldBuffer &hb, uint32_t cur, hipStream_t st)
{
    const uint32_t packed = src == kWaitingUpdates ? 1u : 0u;
    const uint32_t *n_dev = packed ? &hdr->n_batch : nullptr;
    const uint32_t ntiles = (n + kHoldTile - 1) / kHoldTile;
    // a caller's batch appends to the list in use; a replay reads it and builds the other one
    unsigned long long *list_out = packed ? hb.list[cur ^ 1u] : hb.list[cur];
    hipLaunchKernelGGL(hold_count_kernel, dim3(ntiles), dim3(kHoldThreads), 0, st, keys, n, n_dev, g.rows, g.dk, g.dS, rv,
                       packed, tile_count);
    hipLaunchKernelGGL(hold_scan_kernel, dim3(1), dim3(1024), 0, st, tile_count, ntiles, hdr, n, n_dev, packed, hb.cap);
    hipLaunchKernelGGL(hold_scatter_kernel, dim3(ntiles), dim3(kHoldThreads), 0, st, keys, grads, n, n_dev, g.rows, g.D, g.dk,
                       g.dS, rv, packed, tile_count, hdr, list_out, hb.rows, hb.free_list);
    hipLaunchKernelGGL(hold_commit_kernel, dim3(1), dim3(64), 0, st, hdr, packed);
}

void launch_hold_tiles(Header *hdr, const uint32_t *tile_state, const Geometry &g, const RecoveryView &rv, const uint64_t *keys,
                       const float *grads, uint32_t n, BatchSource src, const HoldBuffer &hb, uint32_t cur, hipStream_t st)
{
    const BucketPlan p = bucket_plan(n);
    HoldArgs a;
    a.keys = keys; a.grads = grads; a.tile_state = tile_state;
    a.n = n; a.tiles = p.tiles; a.rows = g.rows; a.packed = src == kWaitingUpdates ? 1u : 0u; a.cap = hb.cap;
    a.geo = g; a.d4 = make_divider(g.D / 4u); a.rv = rv; a.hdr = hdr;
    a.list_out = a.packed ? hb.list[cur ^ 1u] : hb.list[cur];
    a.pool = hb.rows; a.free_list = hb.free_list;
    const dim3 grid(p.tiles), block(kPartThreads);
    switch (p.ipt) {
        case 1: hipLaunchKernelGGL(hold_tiles_kernel<1>, grid, block, 0, st, a); break;
        case 2: hipLaunchKernelGGL(hold_tiles_kernel<2>, grid, block, 0, st, a); break;
        default: hipLaunchKernelGGL(hold_tiles_kernel<4>, grid, block, 0, st, a); break;
    }
}

}  // namespace ecrm
