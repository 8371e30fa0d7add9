"""A bucket's list in LDS around the lengths where its sorting changes: 64 items that a wave counts, 128 that the workgroup counts,
512 that are looked up in one go, the lists of 512 that are merged, and the longest that LDS takes; and around the 64 rows up to
which a list of more than 256 items is sorted by counting.  Entries get several updates each, so that a place that is off by one shows in their arrival
order.  And lists of few stripes, which are cut into a part for each wave at entries: around the 16 items from which on and the 128
up to which they are, the 16 stripes from which on they are not, runs that fill a step, a part or a window, stripes that go on
over two to four parts, and stripes longer than a window, of few entries, which are not cut, and of many; on tables of up
to 16 stripes for a bucket, and on one of more, whose lists are not cut."""
import numpy as np
import pytest

import bucket_plan as bp
from ecrm_case import Case, grads_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n_rows", [(m, max(m // 3, 1)) for m in (1, 2, 63, 64, 65, 127, 128, 129, 192, 511, 512, 513, 576, 1024, 1025,
                                                                   1087, 1535, bp.bucket_cap())] +
                         [(129, 1), (150, 2), (150, 63), (256, 12), (256, 64), (257, 12), (257, 64), (257, 65), (500, 64), (501, 65), (bp.bucket_cap(), 64), (bp.bucket_cap(), 65)])
def test_list_lengths(m, n_rows):
    n, k, S, D, stripes = 6000, 4, 5, 12, 1 << 18
    g = np.arange(stripes, dtype=np.uint32)
    mine = bp.bucket_of(g, n) == 7
    rng = np.random.default_rng(m)
    rows = (rng.permutation(g[mine])[:, None] * k + np.arange(k)).ravel()[:n_rows]
    keys = np.concatenate([rows, rng.choice(rows, m - n_rows), rng.choice(g[~mine], n - m) * k + rng.integers(0, k, n - m)])
    keys = rng.permutation(keys).astype(np.uint64)
    assert len(rows) == n_rows and len(bp.hot_stripes(keys, k)) == 0
    c = Case(k * stripes, D, k, S, max_batch=n, seed=61)
    for call in range(2):
        c.update(keys, grads_for(61, call * n, n, D))
    c.compare(f"list of {m}")


def _few_stripes(k):
    """Lists as runs of (stripe, entry): lengths."""
    rng = np.random.default_rng(k)
    lists = [[[m]] for m in (16, 17, 31, 33, 64)]                                       # one entry
    lists += [[[m // k + (j < m % k) for j in range(k)]] for m in (16, 17, 40, 64, 65, 100, 127, 128, 129, 191, 192, 193)]      # one stripe
    lists += [[[32] * min(k, 4), [1]], [[33] + [1] * (k - 1), [32], [31]], [[1], [62], [1]], [[4] * k] * 4, [[5] * k] * 3, [[1], [30], [30], [30]]]
    for stripes in (2, 3, 4, 5, 14, 15, 16, 17):
        for top in (2, 5, 9, 24):
            runs = [[int(v) for v in rng.integers(1, top, rng.integers(1, k + 1))] for _ in range(stripes)]
            lists.append(runs)
    return [r for r in lists if sum(map(sum, r)) <= 200]


@pytest.mark.parametrize("opt,comb,prop", [(0, 0, 0), (1, 0, 0), (0, 1, 0), (1, 1, 0), (0, 0, 2)])
@pytest.mark.parametrize("D,k,stripes", [(12, 4, 15999), (12, 4, 16000), (128, 5, 15999), (132, 4, 15999), (516, 3, 15999), (36, 63, 15999)])
def test_lists_of_few_stripes(D, k, stripes, opt, comb, prop):
    n, S = 8000, max(7, k + 1)
    assert bp.lists_are_cut(stripes, n) == (stripes < 16000)
    g = np.arange(stripes, dtype=np.uint32)
    bucket = bp.bucket_of(g, n)
    rng = np.random.default_rng(D)
    keys, lists = [], _few_stripes(k)
    chosen = np.argsort(-np.bincount(bucket.astype(np.int64)), kind="stable")[:len(lists)]      # buckets of 17 stripes at least
    for b, runs in zip(chosen, lists):
        for s, entries in zip(np.sort(rng.choice(g[bucket == b], len(runs), replace=False)), runs):
            for j, m in zip(np.sort(rng.choice(k, len(entries), replace=False)), entries):
                keys.append(np.full(m, s * k + j))
    keys = np.concatenate(keys)
    others = g[~np.isin(bucket, chosen)]
    keys = np.concatenate([keys, rng.choice(others, n - len(keys)) * k + rng.integers(0, k, n - len(keys))])
    keys = next(p for p in (rng.permutation(keys).astype(np.uint64) for _ in range(99)) if not len(bp.hot_stripes(p, k)))
    c = Case(k * stripes, D, k, S, max_batch=n, seed=62, optimizer=opt, momentum=0.9, combine=comb, propagation=prop)
    for call in range(2):
        c.update(keys, grads_for(62, call * n, n, D))
    c.compare(f"few stripes {(D, k, opt, comb, prop)}")


@pytest.mark.parametrize("opt,comb", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("D,k", [(12, 4), (128, 4), (260, 4), (128, 10)])
def test_a_short_list_before_another_one_of_its_bucket(D, k, opt, comb):
    """Buckets of more items than LDS takes, which are worked off in parts: a list that is cut at entries comes first, and what it
    leaves in LDS has to be there until all waves are done with it, though the workgroup goes on to the next list."""
    n, stripes, shape = 40000, 16383, [15] * 4 + [200] * 8
    assert bp.lists_are_cut(stripes, n)
    g = np.arange(stripes, dtype=np.uint32)
    bucket, low = bp.bucket_of(g, n).astype(np.int64), bp.scramble(g) & 3
    rng = np.random.default_rng(D + k)
    keys = []
    buckets = np.nonzero(np.min([np.bincount(bucket[low == v], minlength=bp.buckets(n)) for v in (0, 1, 3)], axis=0) >= 4)[0][:20]
    assert len(buckets) == 20
    for b in buckets:
        mine = g[bucket == b]
        chosen = np.concatenate([mine[low[bucket == b] == v][:4] for v in (0, 1, 3)])
        assert [len(l) for l in bp.oversized_parts(chosen, shape, k)] == [4, 4, 4]
        keys.append(np.repeat(chosen, shape) * k + rng.integers(0, k, sum(shape)))
    keys = np.concatenate(keys)
    others = g[~np.isin(bucket, buckets)]
    at = rng.permutation(np.setdiff1d(np.arange(n), bp.sample_positions(n)))[:len(keys)]        # none of them is seen to be hot
    batch = rng.choice(others, n) * k + rng.integers(0, k, n)
    batch[at] = keys
    assert not len(bp.hot_stripes(batch, k))
    c = Case(k * stripes, D, k, 11, max_batch=n, seed=63, optimizer=opt, momentum=0.9, combine=comb)
    for call in range(2):
        c.update(batch.astype(np.uint64), grads_for(63, call * n, n, D))
    c.compare(f"short list before another {(D, k, opt, comb)}")
