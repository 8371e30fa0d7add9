"""The apply kernels of the large batches against the oracle where they can go wrong: row widths around the slices of 128
floats, the order of the list of groups (stripes around the 256 updates above which a stripe is walked first), runs and
stripes around the 64 positions a wave looks at, with the list (more than 2^18 updates) and without, every rule, with and
without parities.  Tolerance: that of Case.compare (fp64 chains rounded once on both sides)."""
import numpy as np
import pytest

import synth_inputs as si
from ecrm_case import Case, grads_for, log

pytestmark = pytest.mark.gpu

LIST = (1 << 18) + 1


@pytest.mark.parametrize("opt,comb,prop", [(0, 0, 0), (1, 0, 0), (0, 1, 0), (1, 1, 0), (0, 0, 2)])
@pytest.mark.parametrize("D,k,S,n", [(4, 1, 2, LIST), (20, 3, 5, LIST), (32, 10, 11, LIST + 4095), (36, 4, 5, LIST), (64, 2, 5, LIST + 17),
                                     (64, 4, 70, 9000), (24, 2, 66, 9001), (68, 4, 5, LIST), (200, 2, 3, LIST)])
def test_widths_and_long_stripes(D, k, S, n, opt, comb, prop):
    rng = np.random.default_rng(D + n)
    R = k * (n // 6)
    lens = [1, 2, 15, 16, 17, 47, 48, 49, 63, 64, 65, 241, 255, 256, 257, 258, 272, 513]
    if n >= LIST:
        lens += [1023, 1024, 1025, 2500]
    stripes = rng.permutation(R // k)[:2 * len(lens)]
    stripes[0] = R // k - 1                                                     # one of them at the batch's end
    keys = []
    for i, m in enumerate(lens[::-1]):
        keys.append(np.full(m, stripes[2 * i] * k + i % k))                     # one entry has all of a stripe's updates
        keys.append(stripes[2 * i + 1] * k + rng.integers(0, k, m))             # ... or its entries share them
    keys = np.concatenate(keys)
    keys = rng.permutation(np.concatenate([keys, rng.integers(0, R, n - len(keys))])).astype(np.uint64)
    c = Case(R, D, k, S, max_batch=n, seed=91, optimizer=opt, momentum=0.9, combine=comb, propagation=prop)
    c.ctx.tune(1, 0xFFFFFFFF)                                                   # ECRM_TUNE_MID_MIN_ROWS: not through buckets
    g = grads_for(91, 0, n, D)
    c.update(keys, g)
    c.update(keys[::-1].copy(), g)
    log("widths", (D, k, S, n, opt, comb, prop), c.compare("widths"))
    if prop == 0:
        c.check_invariant()
