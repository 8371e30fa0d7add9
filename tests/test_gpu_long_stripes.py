"""Stripes that a workgroup's waves share: runs around the 32 updates from which on the waves share a run's columns (eight
updates to a group of lanes, 32 to a round) and the length from which on one leaves its bucket for heavy_stripes, beside runs
that one wave takes as a whole, rows that end inside a wave's 32 columns, and the smallest buckets."""
import numpy as np
import pytest
import torch

import bucket_plan as bp
import synth_inputs as si
from ecrm_case import Case, grads_for
from test_gpu_hold_tiles import _both, _start

pytestmark = pytest.mark.gpu

LEAVES = bp.heavy_run(4000)                              # of a batch of this size
LENS = [[58, 1], [31, 32, 33, 1], [127], [65, 40, 3, 96], [8, 39, 40, 41], [5] * 12, [64, 64], [126, 2, 1, 33], [128, 129],
        [192, 3, 1, 70], [224, 225], [LEAVES - 1], [LEAVES], [LEAVES, 3 * LEAVES // 4]]


@pytest.mark.parametrize("D,k,S", [(4, 4, 5), (36, 12, 13), (128, 4, 5), (132, 4, 5), (260, 12, 13), (1024, 4, 5)])
@pytest.mark.parametrize("opt,comb,prop", [(0, 0, 0), (1, 0, 0), (0, 1, 0), (1, 1, 2), (0, 0, 2)])
def test_shared_stripes(D, k, S, opt, comb, prop):
    R = k * 3000
    rng = np.random.default_rng(7)
    keys = []
    for g, lens in enumerate(LENS):
        lens = lens[:k] if len(lens) > k else lens
        for j, m in enumerate(lens):
            keys += [(g * 211 + 5) * k + j] * m
    taken = [g * 211 + 5 for g in range(len(LENS))]
    rest = rng.choice(np.setdiff1d(np.arange(R // k), taken), 1000) * k
    keys = rng.permutation(np.concatenate([keys, rest])).astype(np.uint64)
    assert len(keys) < 4096 and bp.heavy_run(len(keys)) == LEAVES           # no sample is taken: nothing is known beforehand
    c = Case(R, D, k, S, max_batch=len(keys), seed=91, optimizer=opt, momentum=0.9, combine=comb, propagation=prop)
    for call in range(2):
        c.update(keys, grads_for(91, call * len(keys), len(keys), D))
    left = int(c.scratch[:256].cpu().numpy().view(np.uint32)[22])           # stripes that heavy_stripes was left
    assert left == 2
    c.compare("shared stripes")


@pytest.mark.parametrize("n", [1, 3, 7, 8, 9, 15, 16, 17, 31, 33, 63, 65, 1023])
def test_smallest_buckets(n):
    R, D, k, S = 4 * 64, 64, 4, 5
    c = Case(R, D, k, S, max_batch=n, seed=92)
    for call in range(2):
        c.update(si.uniform_keys(92, call * n, n, R), grads_for(92, call * n, n, D))
    c.compare("smallest buckets")


@pytest.mark.parametrize("n", [1, 7, 8, 9, 16, 17, 33, 65, 1023, 3072])
def test_smallest_buckets_during_a_recovery(n):
    """Without one so few updates take a single launch."""
    R, D, k, S, server = 4 * 64, 64, 4, 5, 3
    c, ses = _start(n, R, D, k, S, server, 6 * n)
    for call in range(4):
        if call % 2:
            c.ctx.recovery_lock(); ses.lock()
        assert _both(c, ses, si.uniform_keys(94, call * n, n, R), grads_for(94, call * n, n, D))
        if call % 2:
            c.ctx.recovery_decode(); ses.decode()
            c.ctx.recovery_unlock(); ses.unlock()
        assert c.ctx.recovery_state()["buffered"] == len(ses.buf_keys)
    assert not c.ctx.recovery_state()["active"]
    c.compare("smallest buckets during a recovery")


@pytest.mark.parametrize("others", [0, 3400])               # in one launch, through the buckets
def test_infinities_in_a_shared_run(others):
    """What an infinity or a NaN among the gradients of a long run makes of its column, and of no other."""
    R, D, k, S, n = 4 * 100, 36, 4, 5, 100
    rest = np.random.default_rng(93).integers(4 * 20, R, others)
    keys = np.concatenate([np.full(n, 41), np.full(60, 42), rest]).astype(np.uint64)
    for opt in (0, 1):
        c = Case(R, D, k, S, max_batch=len(keys), seed=93, optimizer=opt, momentum=0.9)
        g = grads_for(93, 0, len(keys), D)
        g[50, 3], g[3, 7], g[130, 9] = float("inf"), float("nan"), float("-inf")
        c.update(keys, g)
        for t, h in ((c.E, c.hE), (c.A, c.hA)):
            got = t.cpu().numpy()
            np.testing.assert_array_equal(np.isnan(got), np.isnan(h))
            np.testing.assert_array_equal(np.isinf(got), np.isinf(h))
            fine = np.isfinite(h)
            np.testing.assert_allclose(got[fine], h[fine], rtol=1e-5, atol=1e-9 if h is c.hA else 5e-7)
