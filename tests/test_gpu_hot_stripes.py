"""Hot stripes around the sizes up to which they are worked off beside the buckets: one update fewer and more than that limit,
whole rounds of 256 updates and their remainders, an entry with one update beside one with thousands, and the numbers of members
(16) up to which it is done.  The library's own sample says that the stripes are hot."""
import numpy as np
import pytest
import torch

import bucket_plan as bp
from ecrm_case import Case, grads_for

pytestmark = pytest.mark.gpu


def _batch(n, R, k, hot, seed):
    """n keys, hot: {row: number of updates}, the rest uniform over the other stripes"""
    rng = np.random.default_rng(seed)
    stripes = {x // k for x in hot}
    others = np.array([g for g in range(R // k) if g not in stripes])
    m = n - sum(hot.values())
    rest = rng.choice(others, m) * k + rng.integers(0, k, m)
    keys = rng.permutation(np.concatenate([np.repeat(list(hot), list(hot.values())), rest])).astype(np.uint64)
    found = set(bp.hot_stripes(keys, k).tolist())
    assert stripes <= found, "the sample is meant to find them"
    return keys


@pytest.mark.parametrize("total", [900, 1024, 2047, 2048, 2049, 3000])
@pytest.mark.parametrize("D,k,S,opt,comb,prop", [(128, 4, 5, 0, 0, 0), (36, 3, 4, 1, 0, 0), (260, 4, 5, 0, 1, 0), (20, 2, 5, 1, 1, 2),
                                                 (128, 16, 17, 0, 0, 0), (64, 17, 18, 0, 0, 2)])
def test_limits(total, D, k, S, opt, comb, prop):
    n, R = 12000, k * 900
    hot = {7 * k: total - 257, 7 * k + 1: 256, 8 * k + k - 1: 600}
    if k > 2:
        hot[7 * k] -= 1
        hot[7 * k + 2] = 1
    keys = _batch(n, R, k, hot, total)
    c = Case(R, D, k, S, max_batch=n, seed=94, optimizer=opt, momentum=0.9, combine=comb, propagation=prop)
    for call in range(2):
        c.update(keys, grads_for(94, call * n, n, D))
    c.compare("hot stripes")


def test_limit_of_a_large_batch():
    """n / 16 updates in place, one more left to heavy_stripes; three stripes of each kind"""
    n, k, S, D = 200000, 4, 5, 8
    R = k * 20000
    hot = {k * (50 + i): n // 16 + (i % 2) for i in range(6)}
    keys = _batch(n, R, k, hot, 5)
    c = Case(R, D, k, S, max_batch=n, seed=95)
    for call in range(2):
        c.update(keys, grads_for(95, call * n, n, D))
    c.compare("large batch")
    assert c.ctx.batch_stats() is not None
