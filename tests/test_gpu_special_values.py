"""Infinities, NaN and signed zeros in entries, state, parities and gradients: every path through the update has to give
what the rule gives when it is applied update by update in 64 bits, with the differences added to the parities once per
call.  Runs from one update to more than the 128 above which a workgroup walks a stripe.  In one launch, through the buckets -- without
a sample for hot stripes, with some worked off beside the buckets, with a run that is cut into segments -- and through the sort (the
tuning knob sends a batch there)."""
import numpy as np
import pytest
import torch

import bucket_plan as bp
import synth_inputs as si
from ecrm_case import RTOL, Case, grads_for

pytestmark = pytest.mark.gpu

LENS = [1, 2, 3, 4, 5, 7, 8, 9, 31, 63, 64, 65, 127, 128, 129, 300, 600]
PATHS = {"direct": 0, "sort": 0, "buckets": 2000, "hot": 8000, "segments": 2500}       # path: updates on other rows
RULES = [(0, 0, 0.0), (0, 1, 0.0), (1, 0, 0.9), (1, 1, 0.9), (1, 0, 0.001), (1, 0, 0.0)]


def reference(tables, keys, grads, k, lr, eps, opt, comb, mu):
    """The rule applied update by update: tables as stored, results in 64 bits."""
    E, A, PE, PA = (t.astype(np.float64) for t in tables)
    lr, eps, mu = (float(np.float32(v)) for v in (lr, eps, mu))
    for x in np.unique(keys):
        a0, acc = A[x].copy(), np.zeros(E.shape[1])
        gs = grads[keys == x].astype(np.float64)
        if comb:
            total = np.zeros(E.shape[1])
            for g in gs:
                total = total + g
            gs = total[None]
        a = a0.copy()
        for g in gs:
            a = a + g * g if opt == 0 else mu * a + g
            acc = acc + (lr * g / np.sqrt(a + eps) if opt == 0 else lr * a)
        A[x] = a
        E[x] = E[x] - acc
        PE[x // k] = PE[x // k] - acc
        PA[x // k] = PA[x // k] + (a - a0)
    return E, A, PE, PA


def run(D, opt, comb, mu, path, spoil):
    """One call on tables and gradients that spoil(tables, keys, grads) has put its values into; compares all tables."""
    k, S, R = 4, 5, 4 * 64 if PATHS[path] == 0 else 4 * 2000
    keys = np.concatenate([np.full(m, 4 * i + i % 4) for i, m in enumerate(LENS)] + [[4 * 40 + 1, 4 * 40 + 2, 4 * 40 + 2]])
    rng = np.random.default_rng(13)
    keys = np.concatenate([keys, rng.integers(4 * 64, R, PATHS[path]) if PATHS[path] else [], np.full(8300 if path == "segments" else 0, 4 * 50)])
    keys = rng.permutation(keys).astype(np.uint64)
    n = len(keys)
    assert (n <= bp.direct_batch()) == (path in ("direct", "sort")) and (bp.buckets(n) * 16 > R // k) and (path != "buckets" or n < 4096)
    if path == "hot":
        assert bp.divide_hot(keys, k, D)[0]
    if path == "segments":
        assert np.bincount(keys.astype(np.int64) // k).max() >= bp.split_stripe(n, D)
    c = Case(R, D, k, S, max_batch=n, seed=83, optimizer=opt, momentum=mu, combine=comb)
    if path == "sort":
        c.ctx.tune(1, 0xFFFFFFFF)                   # ECRM_TUNE_MID_MIN_ROWS: not through buckets
    tables = [t.cpu().numpy().copy() for t in (c.E, c.A, c.PE, c.PA)]
    grads = grads_for(83, 0, n, D).cpu().numpy().copy()
    spoil(tables, keys, grads)
    for t, h in zip((c.E, c.A, c.PE, c.PA), tables):
        t.copy_(torch.from_numpy(h))
    with np.errstate(all="ignore"):
        want = reference(tables, keys, grads, k, si.DEFAULT_LR, si.DEFAULT_EPS, opt, comb, mu)
    c.ctx.update(torch.from_numpy(keys.view(np.int64)).cuda(), torch.from_numpy(grads).cuda())
    assert c.ctx.status() == 0
    for name, got, w in zip("E A PE PA".split(), (c.E, c.A, c.PE, c.PA), want):
        got, w = got.cpu().numpy(), w.astype(np.float32)
        ordinary = np.isfinite(w) & (w != 0)
        np.testing.assert_array_equal(np.isnan(got), np.isnan(w), err_msg=name)
        np.testing.assert_array_equal(got[np.isinf(w)], w[np.isinf(w)], err_msg=name)
        np.testing.assert_allclose(got[ordinary], w[ordinary], rtol=RTOL, atol=5e-7, err_msg=name)
        yield name, got, w


def middle(keys):
    """Position of the middle update of every row's run."""
    return np.array([np.nonzero(keys == x)[0][(keys == x).sum() // 2] for x in np.unique(keys)])


@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("D", [8, 260])
@pytest.mark.parametrize("opt,comb,mu", RULES[:4])
def test_infinities(opt, comb, mu, D, path):
    def spoil(tables, keys, grads):
        E, A, PE, PA = tables
        grads[middle(keys), 0] = np.inf
        grads[middle(keys), D - 1] = np.nan
        grads[middle(keys)[::2], 1] = -np.inf
        E[:, 2] = -np.inf
        PE[:, 2] = -np.inf
        PE[:, 3] = np.inf
        PA[:, 3] = np.inf
        if opt == 1:
            A[:, 5] = -np.inf                       # an Adagrad accumulator is a sum of squares: never infinite before NaN
    for name, got, w in run(D, opt, comb, mu, path, spoil):
        assert np.isinf(w).any()


@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("D", [8, 260])
@pytest.mark.parametrize("opt,comb,mu", RULES)
def test_signed_zeros(opt, comb, mu, D, path):
    def spoil(tables, keys, grads):
        E, A, PE, PA = tables
        E[:, :4] = -0.0
        PE[:, :3] = -0.0
        PA[:, :2] = -0.0
        grads[:, 0] = 0.0
        grads[:, 1:3] = -0.0
        if opt == 1:
            A[:, :3] = -0.0
    for name, got, w in run(D, opt, comb, mu, path, spoil):
        zero = w == 0
        assert zero.any() or (name == "A" and opt == 0)       # Adagrad's accumulators start above zero
        np.testing.assert_array_equal(got[zero], 0.0, err_msg=name)
        np.testing.assert_array_equal(np.signbit(got[zero]), np.signbit(w[zero]), err_msg=name)


@pytest.mark.parametrize("path", [p for p in PATHS if p != "sort"])
@pytest.mark.parametrize("mu", [0.001, 1e-20, 0.0])
def test_infinite_velocity_under_a_strong_decay(mu, path):
    """Heavy stripes: the decay over 128 updates underflows in 64 bits, but the rule keeps an infinite velocity infinite
    (with mu = 0 it makes NaN of it at the next update)."""
    def spoil(tables, keys, grads):
        tables[1][:, 0] = -np.inf
        grads[middle(keys), 1] = np.inf
    for name, got, w in run(16, 1, 0, mu, path, spoil):
        assert np.isinf(w).any() or mu == 0
