"""Hot stripes on both sides of what sends them beside the buckets or to heavy_stripes behind them: one update fewer and more than
the size up to which they go beside, in small batches and in large ones; whole rounds of 256 updates and their remainders, an
entry with one update beside one with thousands, and the numbers of members (16) up to which it is done; and batches of so many
that none does, whose entries all of the hot workgroups hand on.  The library's own plan and sample say which way a batch goes,
and the header of the scratch buffer which way it went."""
import numpy as np
import pytest
import torch

import bucket_plan as bp
from ecrm_case import Case, grads_for

pytestmark = pytest.mark.gpu


def _batch(n, R, k, D, hot, seed, here):
    """n keys, hot: {row: number of updates}, the rest uniform over the other stripes; in an order in which the sample sends
    exactly the stripes `here` beside the buckets"""
    rng = np.random.default_rng(seed)
    stripes = {x // k for x in hot}
    others = np.array([g for g in range(R // k) if g not in stripes])
    m = n - sum(hot.values())
    rest = rng.choice(others, m) * k + rng.integers(0, k, m)
    keys = np.concatenate([np.repeat(list(hot), list(hot.values())), rest]).astype(np.uint64)
    for _ in range(400):
        keys = rng.permutation(keys)
        if bp.divide_hot(keys, k, D)[0] == here:
            return keys
    raise AssertionError("no such order found")


def _header(c):
    """heavy_run, the bits of the stripes that were to go beside the buckets, and what heavy_stripes was left: stripes, segments"""
    w = c.scratch[:256].cpu().numpy().view(np.uint32)
    return int(w[29]), int(w[30]) | int(w[31]) << 32, int(w[22]), int(w[24])


def _twice(c, keys, seed):
    n, D = len(keys), c.D
    for call in range(2):
        c.update(keys, grads_for(seed, call * n, n, D))
    return _header(c)


@pytest.mark.parametrize("total", [769, 770, 1025, 2047, 2048, 2049, 3000])
@pytest.mark.parametrize("D,k,S,opt,comb,prop", [(128, 4, 5, 0, 0, 0), (36, 3, 4, 1, 0, 0), (260, 4, 5, 0, 1, 0), (20, 2, 5, 1, 1, 2),
                                                 (128, 16, 17, 0, 0, 0), (64, 17, 18, 0, 0, 2)])
def test_limits(total, D, k, S, opt, comb, prop):
    """Stripe 7 has `total` updates, 256 of them in one entry; 512 and 513 are among the longest runs."""
    n, R = 12000, k * 900
    limit = bp.hot_in_place(n)
    assert limit == 2048
    hot = {7 * k: total - 256, 7 * k + 1: 256, 8 * k + k - 1: 600}
    if k > 2:
        hot[7 * k] -= 1
        hot[7 * k + 2] = 1
    # as the sample sees it; the exact size is looked at again, where it is known
    here = set() if k > 16 else {7, 8} if total <= limit + 1 else {8}
    keys = _batch(n, R, k, D, hot, total, here)
    assert np.bincount(keys.astype(np.int64) // k)[7] == total
    c = Case(R, D, k, S, max_batch=n, seed=94, optimizer=opt, momentum=0.9, combine=comb, propagation=prop)
    heavy_run, bits, stripes, segments = _twice(c, keys, 94)
    ranked = [g for g, _, _ in bp.ranked_hot_stripes(keys, k)[0]]
    assert {g for i, g in enumerate(ranked) if bits >> i & 1} == here
    assert segments == 0 and stripes == (2 if k > 16 else 1 if total > limit else 0)
    assert heavy_run == (128 if (total == 3000 or k > 16) and D <= 128 else 256)     # shorter where heavy_stripes has work anyway
    c.compare("hot stripes")


@pytest.mark.parametrize("D", [128, 260])
def test_limit_of_a_large_batch(D):
    """n / 16 updates, one fewer and one more; and a stripe of twice as many, which is always left"""
    n, k, S = 200000, 4, 5
    R, limit = k * 20000, bp.hot_in_place(200000)
    assert limit == n // 16 and limit + 1 < bp.split_stripe(n, D)
    sizes = {50: limit - 1, 51: limit, 52: limit + 1}
    keys = _batch(n, R, k, D, {k * g + g % k: m for g, m in sizes.items()}, 5, set(sizes))
    count = np.bincount(keys.astype(np.int64) // k)
    assert all(count[g] == m for g, m in sizes.items())
    c = Case(R, D, k, S, max_batch=n, seed=95)
    heavy_run, _, stripes, segments = _twice(c, keys, 95)
    assert (stripes, segments) == (1, 0) and heavy_run == bp.heavy_run(n)
    stats = c.ctx.batch_stats()
    assert stats["long_rows"] == 3 and stats["long_items"] == sum(sizes.values())
    c.compare("large batch")


@pytest.mark.parametrize("k,D", [(4, 128), (2, 512), (1, 20), (10, 64), (37, 36)])
def test_handed_on(k, D):
    """More hot stripes than are numbered, or as many as there are: every entry is copied for heavy_stripes, or described to it if
    its stripe is among the longest."""
    n, S = 1 << 15, k + 1
    R = k * 24
    rng = np.random.default_rng(k)
    keys = np.concatenate([rng.integers(0, R, n - 9000), rng.integers(0, k, 9000)])
    keys = rng.permutation(keys).astype(np.uint64)
    here, left = bp.divide_hot(keys, k, D)
    assert not here and left
    c = Case(R, D, k, S, max_batch=n, seed=96)
    heavy_run, bits, stripes, segments = _twice(c, keys, 96)
    described = int(np.bincount(keys.astype(np.int64) // k)[0] >= bp.split_stripe(n, D))
    assert bits == 0 and stripes == min(24, 256 // k) - described and (segments > 0) == bool(described)
    c.compare("handed on")
