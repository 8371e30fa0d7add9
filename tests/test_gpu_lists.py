"""A bucket's list in LDS around the lengths where its sorting changes: 64 items that a wave counts, 128 that the workgroup counts,
512 that are looked up in one go, the lists of 512 that are merged, and the longest that LDS takes; and around the 64 rows up to
which a list is sorted by counting.  Entries get several updates each, so that a place that is off by one shows in their arrival
order."""
import numpy as np
import pytest

import bucket_plan as bp
from ecrm_case import Case, grads_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n_rows", [(m, max(m // 3, 1)) for m in (1, 2, 63, 64, 65, 127, 128, 129, 192, 511, 512, 513, 576, 1024, 1025,
                                                                   1087, 1535, bp.bucket_cap())] +
                         [(129, 1), (150, 2), (150, 63), (500, 64), (501, 65), (bp.bucket_cap(), 64), (bp.bucket_cap(), 65)])
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
