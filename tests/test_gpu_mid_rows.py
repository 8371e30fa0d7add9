"""Batches with enough long entries that one workgroup walks many of them while the first pass over the others' pieces goes on in
the same launch: entries on both sides of that limit, rows of one and of two slices a lane, and one batch just short of it."""
import numpy as np
import pytest
import torch

from ecrm_case import Case, grads_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,k,long_rows", [(100, 4, 430), (68, 10, 410), (132, 2, 401), (68, 4, 399), (8, 4, 450)])
def test_runs_and_pieces_together(D, k, long_rows):
    S, R = k + 1, k * 20000
    rng = np.random.default_rng(D)
    rows = rng.permutation(R)[:long_rows]
    lens = rng.integers(1025, 1200, long_rows)
    limit = 12 * long_rows
    lens[:6] = [limit, limit + 1, 9000, 4 * limit // 3, 1025, limit - 1]
    others = np.setdiff1d(np.arange(R), rows)                        # the lengths are exact
    rest = rng.choice(others, max((1 << 21) + 1 - int(lens.sum()), 1000))
    keys = rng.permutation(np.concatenate([np.repeat(rows, lens), rest])).astype(np.uint64)
    n = len(keys)
    assert n > 1 << 21
    counts = np.bincount(keys.astype(np.int64), minlength=R)
    assert (counts[rows] == lens).all() and counts[others].max() <= 1024
    c = Case(R, D, k, S, max_batch=n, seed=101)
    for call in range(2):
        c.update(keys, grads_for(101, call * n, n, D))
        stats = c.ctx.batch_stats()
        long = counts[counts > 1024]
        assert stats["long_rows"] == len(long)
        want = int((long <= 12 * len(long)).sum()) if len(long) >= (400 if D > 64 else 2048) else 0
        assert stats["one_workgroup_rows"] == want and stats["pieces"] > 0
    c.compare("runs and pieces")
