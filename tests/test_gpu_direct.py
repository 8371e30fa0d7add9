"""Batches of up to 3072 updates, which take one launch, against the oracle: sizes around the two variants' 2048 and 3072 keys and
around a workgroup's 256, stripes around the 192 updates from which on they are taken by columns, runs of it around the 32 up to
which a group of lanes takes them, more such stripes than there are workgroups for, rows of more than 1024 updates, every rule; batches of
nothing but stripes of a few hundred updates, which stay in their buckets or make more jobs than the workgroups for them take at once; and
a batch with a bad key, at each place a workgroup reads."""
import numpy as np
import pytest
import torch

import bucket_plan as bp
import synth_inputs as si
from ecrm_case import Case, grads_for

pytestmark = pytest.mark.gpu
RULES = [(0, 0), (1, 0), (0, 1), (1, 1)]


def _check(c, keys, seed, what):
    for call in range(2):
        c.update(keys if call == 0 else keys[::-1].copy(), grads_for(seed, call * len(keys), len(keys), c.D))
    counts = np.bincount(keys.astype(np.int64))
    stats = c.ctx.batch_stats()
    assert stats["long_rows"] == int((counts > 1024).sum())
    assert stats["long_items"] == int(counts[counts > 1024].sum())
    c.compare(what)
    if c.propagation == 0:
        c.check_invariant()


@pytest.mark.parametrize("prop", [0, 2])
@pytest.mark.parametrize("n", [1, 8, 9, 255, 256, 257, 2047, 2048, 2049, 3071, 3072, 3073])
def test_sizes(n, prop):
    R, D, k, S = 4 * 1500, 36, 4, 5
    c = Case(R, D, k, S, max_batch=n, seed=71, propagation=prop)
    _check(c, si.uniform_keys(71, 0, n, R), 71, f"direct {n}")


@pytest.mark.parametrize("opt,comb", RULES)
@pytest.mark.parametrize("D,k,S", [(4, 1, 2), (128, 4, 5), (132, 40, 64), (1024, 63, 64)])
def test_long_stripes(D, k, S, opt, comb):
    R = k * 300
    rng = np.random.default_rng(5)
    stripes = rng.permutation(R // k)[:8]
    keys = [np.full(m, stripes[i] * k + i % k) for i, m in enumerate([bp.direct_long() - 1, bp.direct_long(), 257, 513])]
    shares = [1, 31, 32, 33, 96, 7][:k]                                       # runs of one stripe
    for j, m in enumerate(shares):
        keys.append(np.full(m, stripes[4] * k + j))
    keys.append(stripes[5] * k + rng.integers(0, k, 300))                     # all entries of a stripe, about 5 or 8 updates each
    keys.append(rng.integers(0, R, 900))
    keys = rng.permutation(np.concatenate(keys)).astype(np.uint64)
    assert len(keys) <= bp.direct_batch()
    c = Case(R, D, k, S, max_batch=len(keys), seed=72, optimizer=opt, momentum=0.9, combine=comb)
    _check(c, keys, 72, f"direct long {(D, k, opt, comb)}")


@pytest.mark.parametrize("n", [2048, 3072])
@pytest.mark.parametrize("R,k", [(1, 1), (4, 4), (60, 4), (2, 1)])
def test_nothing_but_long_stripes(R, k, n):
    D, S = 260, k + 1                                                         # 15 stripes of 33 groups of columns; one row of 3072 updates
    c = Case(R, D, k, S, max_batch=n, seed=73)
    _check(c, si.uniform_keys(73, 0, n, R), 73, f"direct few rows {(R, n)}")


@pytest.mark.parametrize("opt,comb", RULES)
@pytest.mark.parametrize("R,k,D,every", [(56, 4, 128, False), (100, 10, 260, False), (140, 10, 32, False), (10, 1, 260, True), (40, 4, 1024, True),
                                         (882, 63, 132, True), (60, 10, 4, False), (12, 4, 1024, True)])
def test_stripes_of_a_few_hundred_updates(R, k, D, every, opt, comb):
    n, S = 3000, k + 1
    keys = si.uniform_keys(75, 0, n, R)
    runs = [np.unique(keys[keys // k == g], return_counts=True)[1].tolist() for g in range(R // k)]
    columns = [bp.direct_by_columns(r, n, R // k, D) for r in runs if sum(r) >= bp.direct_long()]
    assert all(columns) if every else not all(columns)
    c = Case(R, D, k, S, max_batch=n, seed=75, optimizer=opt, momentum=0.9, combine=comb)
    _check(c, keys, 75, f"direct, a few hundred {(R, k, D, opt, comb)}")


@pytest.mark.parametrize("n,at", [(1, 0), (600, 599), (2048, 2047), (3072, 1300)])
def test_a_bad_key_rejects_the_batch(n, at):
    R, D, k, S = 4 * 500, 128, 4, 5
    c = Case(R, D, k, S, max_batch=n, seed=74)
    keys = si.uniform_keys(74, 0, n, R)
    bad = keys.copy()
    bad[at] = R
    before = [t.clone() for t in (c.E, c.A, c.PE, c.PA, c.ld, c.lp)]
    g = grads_for(74, 0, n, D)
    c.ctx.update(torch.from_numpy(bad.view(np.int64)).cuda(), g)
    assert c.ctx.status() == -5
    assert all(torch.equal(x, y) for x, y in zip(before, (c.E, c.A, c.PE, c.PA, c.ld, c.lp)))
    c.ctx.clear_status()
    c.update(keys, g)
    c.compare("after a bad batch")
