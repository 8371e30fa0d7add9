"""Rows of at most 64 floats in the apply kernel of large batches, several of them to a wave: every width around the groups of 16
and 32 lanes, stripes that begin and end anywhere in a step of two or four entries, entries of one to forty updates beside each
other, and with and without parities.  Through the sort (the tuning knob sends a batch there)."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from ecrm_case import Case, grads_for

pytestmark = pytest.mark.gpu

WIDTHS = [4, 8, 12, 28, 32, 36, 40, 60, 64, 68]


def _case(R, D, k, S, n, **kw):
    c = Case(R, D, k, S, max_batch=n, seed=96, **kw)
    c.ctx.tune(1, 0xFFFFFFFF)                        # ECRM_TUNE_MID_MIN_ROWS: not through buckets
    return c


@pytest.mark.parametrize("D", WIDTHS)
@pytest.mark.parametrize("k,S", [(1, 2), (2, 5), (3, 4), (4, 5), (10, 11), (64, 65)])
def test_widths(D, k, S):
    n, R = 6007, k * 700
    rng = np.random.default_rng(D * k)
    c = _case(R, D, k, S, n)
    for call in range(2):
        # uniform, a few entries of up to forty updates, and one whose run leaves the window
        keys = np.concatenate([rng.integers(0, R, n - 1500), np.repeat(rng.integers(0, R, 60), rng.integers(1, 41, 60))[:1400]])
        keys = np.concatenate([keys, np.full(n - len(keys), 5 % R)])
        c.update(rng.permutation(keys).astype(np.uint64), grads_for(96, call * n, n, D))
    c.compare("narrow rows")


@pytest.mark.parametrize("D", [16, 32, 48, 64])
@pytest.mark.parametrize("opt,comb,prop", [(1, 0, 0), (0, 1, 0), (1, 1, 0), (0, 0, 2), (1, 1, 2), (0, 0, 1)])
def test_rules(D, opt, comb, prop):
    n, R, k, S = 20011, 4 * 2000, 4, 5
    c = _case(R, D, k, S, n, optimizer=opt, momentum=0.9, combine=comb, propagation=prop)
    for call in range(2):
        keys = si.uniform_keys(97, call * n, n, R)
        keys[::3] = si.uniform_keys(98, call * n, n, R)[::3] % np.uint64(R // 40)
        c.update(keys, grads_for(97, call * n, n, D))
    c.compare("narrow rules")


@pytest.mark.parametrize("D", [12, 32, 36, 64])
def test_neighbours_are_left_alone(D):
    """Only the rows that are updated change, and only their stripes' parities; the last row of the tables is among them."""
    R, k, S = 4 * 300, 4, 5
    keys = np.array([0, 1, 3, 4, 9, 10, 10, 17, R - 5, R - 1, R - 1], np.uint64)
    c = _case(R, D, k, S, len(keys))
    before = [t.clone() for t in (c.E, c.A, c.PE, c.PA)]
    c.update(keys, grads_for(99, 0, len(keys), D))
    c.compare("neighbours")
    for t, b, rows in zip((c.E, c.A, c.PE, c.PA), before, (keys, keys, keys // 4, keys // 4)):
        left = torch.ones(len(t), dtype=torch.bool, device="cuda")
        left[torch.from_numpy(rows.astype(np.int64)).cuda()] = False
        assert torch.equal(t[left].view(torch.int32), b[left].view(torch.int32))


def test_large_batch():
    """A batch that takes this way by itself."""
    n, R, D, k, S = (1 << 19) + 4099, 2 * 150000, 64, 2, 5
    c = Case(R, D, k, S, max_batch=n, seed=96, optimizer=1, momentum=0.9)
    keys = si.uniform_keys(96, 0, n, R)
    keys[1::2] = si.uniform_keys(95, 0, n, R)[1::2] % np.uint64(500)
    c.update(keys, grads_for(96, 0, n, D))
    c.compare("large batch of narrow rows")
