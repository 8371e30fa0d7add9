"""The sample in which the partition looks for hot stripes, on the host: one position in every segment of the batch, and
blind to no period of it; what becomes of the hot stripes: worked off beside the buckets where that ends with them; and what becomes of the
long stripes of a batch that takes one launch."""
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


def _batch(n, R, k, hot, seed=1):
    """n keys: hot {row: updates}, the rest uniform"""
    rng = np.random.default_rng(seed)
    rest = rng.integers(0, R, n - sum(hot.values()))
    return rng.permutation(np.concatenate([np.repeat(np.array(list(hot), np.int64), list(hot.values())), rest]))


@pytest.mark.parametrize("n,R,k,D", [(1 << 14, 32, 4, 128), (1 << 16, 64, 4, 128), (1 << 16, 128, 4, 512), (1 << 18, 64, 4, 128),
                                     (1 << 18, 256, 4, 512), (1 << 19, 128, 4, 128), (1 << 19, 256, 4, 128)])
def test_a_batch_of_hot_stripes_is_left_to_heavy_stripes(n, R, k, D):
    """Nothing but hot stripes: beside the buckets there is nothing to hide their work behind.  (Worked off there all the same
    they took up to twice as long.)"""
    keys = np.random.default_rng(n + R).integers(0, R, n)
    assert bp.hot_stripes(keys, k).size and bp.divide_hot(keys, k, D) == (set(), True)


@pytest.mark.parametrize("D", [64, 128, 512, 1024])
def test_many_hot_stripes_beside_few_others(D):
    """15 stripes of n / 16 updates in two entries each."""
    for n, k in ((1 << 16, 4), (1 << 17, 4), (1 << 19, 4)):
        hot = {g * k + j: n // 32 for g in range(3, 18) for j in range(2)}
        here, left = bp.divide_hot(_batch(n, n // 2, k, hot), k, D)
        assert left and not here


@pytest.mark.parametrize("n,T", [(8192, 600), (26624, 1500), (65536, 2000), (200000, 6000)])
def test_a_few_hot_stripes_go_beside_the_buckets(n, T):
    k = 4
    hot = {40: T, 81: T // 2, 122: T // 2}
    here, left = bp.divide_hot(_batch(n, 4 * n, k, hot), k, 128)
    assert here == {10, 20, 30} and not left


def test_what_the_sample_says_of_a_stripe():
    u = bp.C.c_uint32
    entries = lambda hits, seen, k: int(bp.lib().plan_sampled_entries(u(hits), u(seen), u(k)))
    assert entries(40, 1, 10) == 1 and entries(40, 4, 4) == 4 and entries(4, 4, 10) == 10 and entries(5, 2, 10) == 3
    for k in (1, 2, 4, 10, 16):
        for hits in range(4, 200):
            for seen in range(1, min(k, hits) + 1):
                assert seen <= entries(hits, seen, k) <= k
    root = lambda v: int(bp.lib().plan_square_root(u(v)))
    assert all(root(v) ** 2 <= v < (root(v) + 1) ** 2 for v in list(range(2000)) + [1 << 21, (1 << 24) - 1])


@pytest.mark.parametrize("n", [4096, 8191, 8192, 65536, 65600, 1 << 19])
@pytest.mark.parametrize("D", [4, 16, 20, 128, 1024])
def test_buckets_beside_hot_stripes(n, D):
    """Without hot stripes all of a plan's buckets are filled; with them those that are resident beside the stripes' workgroups, of
    which there are 192 at most; a plan that leaves them room anyway, or has more buckets than are resident, stays as it is."""
    assert bp.buckets_beside(n, 0, D) == bp.buckets(n)
    for hot in (1, 8, 64):
        beside = 1024 - min(hot * -(-D // 16), 192)
        assert bp.buckets_beside(n, hot, D) == (bp.buckets(n) if bp.buckets(n) > 1024 else min(bp.buckets(n), beside))


def test_no_buckets_stay_empty_for_stripes_that_are_not_beside_them():
    """No stripe of more than 16 entries is worked off beside the buckets, whatever the sample says; and long rows keep all buckets."""
    pays = lambda k, D: bool(bp.lib().plan_beside_pays(bp.C.c_uint32(k), bp.C.c_uint32(D)))
    for k in (1, 4, 16, 17, 63):
        for D in (4, 128, 256, 260, 1024):
            in_place = bool(bp.lib().plan_in_place_size(bp.C.c_uint32(1 << 16), bp.C.c_uint32(k), bp.C.c_uint32(D), bp.C.c_uint32(600)))
            assert in_place == (k <= 16) and pays(k, D) == (in_place and D <= 256)


@pytest.mark.parametrize("D", [32, 128, 256, 512, 1024])
def test_long_stripes_of_a_batch_in_one_launch(D):
    """A stripe with one run goes by columns, and so does any of a thousand updates.  A few hundred updates of several entries alike
    stay in their bucket where the batch is made of such stripes: 3000 updates on 56 and 100 rows took up to 3.5 times as long
    when all of them went by columns."""
    n, by = 3000, bp.direct_by_columns
    assert by([214], n, 14, D) and by([300], n, 10, D) and by([200, 3, 2, 1], n, 1 << 14, D)
    assert by([750] * 4, n, 1, D) and by([250] * 4, n, 3, D) and by([100] * 10, n, 3, D) and by([16] * 63, n, 3, D)
    assert not by([54, 53, 53, 54], n, 14, D) and not by([30] * 6 + [35] * 4, n, 10, D)


@pytest.mark.parametrize("n", [3073, 8192, 65536, 300007, 1 << 19])
def test_lists_are_cut_on_tables_of_some_stripes(n):
    """Neither where most lists have many stripes, nor where the stripes are too long for a list that can be cut."""
    most, least = 16 * bp.buckets(n), n // 88
    assert bp.lists_are_cut(most - 1, n) and not bp.lists_are_cut(most, n)
    assert bp.lists_are_cut(least + 1, n) and not bp.lists_are_cut(least, n) and not bp.lists_are_cut(1, n)
