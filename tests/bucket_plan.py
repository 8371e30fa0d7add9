"""The library's own plan of a batch that goes through buckets, and its sample for hot stripes: csrc/bucket_plan.h compiled
for the host, so that no test has to repeat its formulas."""
from __future__ import annotations

import ctypes as C
import os
import subprocess
import tempfile

import numpy as np

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2104_01981_amd", "csrc")
SOURCE = """
#include "bucket_plan.h"
using namespace ecrm;
extern "C" {
uint32_t plan_buckets(uint32_t n) { return bucket_plan(n).buckets; }
uint32_t plan_buckets_beside(uint32_t buckets, uint32_t hot, uint32_t D) { return buckets_beside(buckets, hot, D); }
uint32_t plan_lists_are_cut(uint32_t stripes, uint32_t n) { return lists_are_cut(stripes, bucket_plan(n).buckets, n); }
uint32_t plan_beside_pays(uint32_t k, uint32_t D) { return beside_pays(k, D); }
uint32_t plan_heavy_run(uint32_t n) { return heavy_run(n); }
uint32_t plan_direct_batch() { return kDirectBatch; }
uint32_t plan_direct_long() { return kDirectLong; }
uint32_t plan_direct_by_columns(uint32_t updates, uint32_t entries, uint32_t longer, uint32_t others, uint32_t third, uint32_t n, uint32_t stripes, uint32_t D)
{
    return direct_by_columns(DirectList{updates, entries, longer, others, third != 0}, n, stripes, D, false);
}
uint32_t plan_bucket_cap() { return kBucketCap; }
uint32_t plan_heavy_stripe(uint32_t k) { return heavy_stripe(k); }
uint32_t plan_split_stripe(uint32_t n, uint32_t D) { return split_stripe(n, D); }
uint32_t plan_shared_stripe(uint32_t n, uint32_t k) { return shared_stripe(n, k); }
uint32_t plan_hot_in_place(uint32_t n) { return hot_in_place(n); }
uint32_t plan_hot_least(uint32_t n, uint32_t k, uint32_t D, uint32_t candidates) { return hot_least(bucket_limits(n, k, D), k, candidates); }
uint32_t plan_many_hot() { return kManyHot; }
uint32_t plan_in_place_size(uint32_t n, uint32_t k, uint32_t D, uint32_t m) { return in_place_size(bucket_limits(n, k, D), k, m); }
uint32_t plan_in_place_time(uint32_t n, uint32_t k, uint32_t D, uint32_t hot, uint32_t rest, uint32_t m0, uint32_t e0, uint32_t m, uint32_t e)
{
    return in_place_time(bucket_limits(n, k, D), D, hot, rest, HotStripe{m0, e0}, HotStripe{m, e});
}
uint32_t plan_sampled_updates(uint32_t hits, uint32_t n) { return sampled_updates(hits, n); }
uint32_t plan_sampled_entries(uint32_t hits, uint32_t seen, uint32_t k) { return sampled_entries(hits, seen, k); }
uint32_t plan_square_root(uint32_t v) { return square_root(v); }
uint32_t plan_hot_hits(uint32_t n) { return hot_hits(n); }
uint32_t plan_sample(uint32_t n, uint32_t *at)
{
    for (uint32_t i = 0; i < 1u << sample_bits(n); ++i) at[i] = sample_position(i, n);
    return 1u << sample_bits(n);
}
void plan_mix(uint32_t *g, uint32_t m) { for (uint32_t i = 0; i < m; ++i) g[i] = mix32(g[i]); }
void plan_scramble(uint32_t *g, uint32_t m) { for (uint32_t i = 0; i < m; ++i) g[i] = scramble32(g[i]); }
}
"""
_lib = None


def lib():
    global _lib
    if _lib is None:
        with tempfile.TemporaryDirectory() as tmp:
            src, out = os.path.join(tmp, "plan.cpp"), os.path.join(tmp, "plan.so")
            with open(src, "w") as f:
                f.write(SOURCE)
            subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-I", CSRC, src, "-o", out])
            _lib = C.CDLL(out)
    return _lib


def buckets(n):
    return int(lib().plan_buckets(C.c_uint32(n)))


def buckets_beside(n, hot, D):
    return int(lib().plan_buckets_beside(C.c_uint32(buckets(n)), C.c_uint32(hot), C.c_uint32(D)))


def heavy_run(n):
    return int(lib().plan_heavy_run(C.c_uint32(n)))


def bucket_cap():
    return int(lib().plan_bucket_cap())


def direct_batch():
    return int(lib().plan_direct_batch())


def direct_long():
    return int(lib().plan_direct_long())


def direct_by_columns(runs, n, stripes, D):
    """Whether the one-launch path has a stripe with these runs worked off by columns (Adagrad)."""
    u, longer = C.c_uint32, [r for r in runs if r >= 32]
    third = max(runs) >= sum(runs) // 3
    return bool(lib().plan_direct_by_columns(u(sum(runs)), u(len(runs)), u(len(longer)), u(sum(runs) - sum(longer)), u(third), u(n), u(stripes), u(D)))


def heavy_stripe(k):
    return int(lib().plan_heavy_stripe(C.c_uint32(k)))


def shared_stripe(n, k):
    return int(lib().plan_shared_stripe(C.c_uint32(n), C.c_uint32(k)))


def split_stripe(n, D):
    return int(lib().plan_split_stripe(C.c_uint32(n), C.c_uint32(D)))


def mix(stripes):
    g = np.ascontiguousarray(stripes, np.uint32).copy()
    lib().plan_mix(g.ctypes.data_as(C.POINTER(C.c_uint32)), C.c_uint32(len(g)))
    return g


def scramble(stripes):
    g = np.ascontiguousarray(stripes, np.uint32).copy()
    lib().plan_scramble(g.ctypes.data_as(C.POINTER(C.c_uint32)), C.c_uint32(len(g)))
    return g


def lists_are_cut(stripes, n):
    return bool(lib().plan_lists_are_cut(C.c_uint32(stripes), C.c_uint32(n)))


def oversized_parts(stripes, updates, k):
    """A bucket of more items than LDS takes, as bucket_apply works it off: one list after the other, each as the numbers of its
    stripes of fewer than heavy_stripe(k) updates.  For buckets of few stripes, which overflow no table."""
    bits, updates, lists = scramble(stripes), np.asarray(updates), []
    assert len(stripes) < 640 and updates.sum() > bucket_cap()

    def walk(part, depth):
        mine = np.nonzero(bits & np.uint32((1 << depth) - 1) == part)[0]
        light = mine[updates[mine] < heavy_stripe(k)]
        if updates[light].sum() > bucket_cap() or len(mine) - len(light) > 16:
            walk(part, depth + 1)
            walk(part | 1 << depth, depth + 1)
        else:
            lists.append(light)

    walk(0, 0)
    return lists


def bucket_of(stripes, n):
    return (mix(stripes).astype(np.uint64) * np.uint64(buckets(n))) >> np.uint64(32)


def sample_positions(n):
    at = np.empty(1024, np.uint32)
    return at[:lib().plan_sample(C.c_uint32(n), at.ctypes.data_as(C.POINTER(C.c_uint32)))].astype(np.int64)


def hot_stripes(keys, k):
    """The stripes that the partition takes for hot (before it keeps the most frequent ones of too many)."""
    g, hits = np.unique(np.asarray(keys, np.int64)[sample_positions(len(keys))] // k, return_counts=True)
    return g[hits >= int(lib().plan_hot_hits(C.c_uint32(len(keys))))]


def hot_in_place(n):
    return int(lib().plan_hot_in_place(C.c_uint32(n)))


def ranked_hot_stripes(keys, k):
    """The stripes of the sample that the partition keeps, as it numbers them: (stripe, hits, of its first 16 entries those seen),
    and how many it had to choose from."""
    sample = np.asarray(keys, np.int64)[sample_positions(len(keys))]
    g, hits = np.unique(sample // k, return_counts=True)
    hot = hits >= int(lib().plan_hot_hits(C.c_uint32(len(keys))))
    g, hits = g[hot], hits[hot]
    order = np.lexsort((g, -hits))[:min(64, 256 // k)]
    seen = [sum(1 for x in np.unique(sample[sample // k == s]) if x % k < 16) for s in g[order]]
    return list(zip(g[order].tolist(), hits[order].tolist(), seen)), len(g)


def divide_hot(keys, k, D):
    """What the partition makes of the hot stripes: those that are worked off beside the buckets, and whether others are left."""
    u, n = C.c_uint32, len(keys)
    ranked, candidates = ranked_hot_stripes(keys, k)
    if n < 4096 or not ranked:
        return set(), False
    updates = [int(lib().plan_sampled_updates(u(h), u(n))) for _, h, _ in ranked]
    entries = [int(lib().plan_sampled_entries(u(h), u(s), u(k))) for _, h, s in ranked]
    rest = n - min(sum(updates), n)
    fits = [bool(lib().plan_in_place_size(u(n), u(k), u(D), u(m))) for m in updates]
    slow = False
    for (_, h, _), e, f in zip(ranked, entries, fits):
        m = lib().plan_sampled_updates(u(h - lib().plan_square_root(u(h))), u(n))
        slow |= f and not lib().plan_in_place_time(u(n), u(k), u(D), u(len(ranked)), u(rest), u(updates[0]), u(entries[0]), u(m), u(e))
    here = set() if slow else {g for (g, _, _), f in zip(ranked, fits) if f}
    least = int(lib().plan_hot_least(u(n), u(k), u(D), u(candidates)))
    return here, any(m >= least and g not in here for (g, _, _), m in zip(ranked, updates))
