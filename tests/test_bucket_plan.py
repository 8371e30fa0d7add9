"""The sample in which the partition looks for hot stripes, on the host: one position in every segment of the batch, and
blind to no period of it."""
import numpy as np
import pytest

import bucket_plan as bp


@pytest.mark.parametrize("n", [4096, 4097, 26624, 65536, 131072, 131073, 300007, 1 << 18, 1 << 19])
def test_one_position_in_every_segment(n):
    at = bp.sample_positions(n)
    edges = np.arange(len(at) + 1, dtype=np.int64) * n // len(at)
    assert (at >= edges[:-1]).all() and (at < edges[1:]).all()


@pytest.mark.parametrize("n", [4096, 26624, 53248, 65536, 1 << 18, 1 << 19])
@pytest.mark.parametrize("period", [2, 3, 4, 8, 13, 16, 26, 32])
def test_every_residue_of_a_period_is_sampled(n, period):
    """Tables that take turns in a batch (position mod period) get their share of the sample: within five standard
    deviations of it, one position per segment drawn evenly.  The length of a segment has to be a period, or it says nothing."""
    at = bp.sample_positions(n)
    if n // len(at) < period:
        pytest.skip("a segment is shorter than the period")
    share = np.bincount(at % period, minlength=period)
    expect = len(at) / period
    assert (np.abs(share - expect) <= 5 * np.sqrt(expect) + 1).all(), share


@pytest.mark.parametrize("n", [26624, 65536, 1 << 18, 1 << 19])
def test_hot_stripes_at_odd_positions_are_found(n):
    """Half of the batch is uniform, the odd positions fall on 8 stripes: each has n / 16 updates."""
    rng = np.random.default_rng(n)
    keys = rng.integers(0, 1 << 20, n)
    keys[1::2] = rng.integers(0, 32, n // 2)
    assert set(range(8)) <= set(bp.hot_stripes(keys, 4).tolist())
