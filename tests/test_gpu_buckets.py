"""The bucket path (batches of up to 2^19 updates) against the oracle where it can go wrong: runs around the 64 positions of a
wave's window and the 128 to 256 updates of a run that may make its stripe heavy, stripes around the lengths from which
they are shared by a workgroup, heavy, or cut into segments, buckets around the 1536 items LDS takes, tiles and bucket
counts at their edges, every rule, row widths with and without a remainder, with and without parities.  Tolerance: that
of Case.compare (fp64 chains rounded once on both sides; a re-association moves a value across a rounding boundary with
probability ~1e-6)."""
import numpy as np
import pytest
import torch

import bucket_plan as bp
import oracle
import synth_inputs as si
from ecrm_case import Case, grads_for, log
from oracle.recovery_session import RecoverySession

pytestmark = pytest.mark.gpu


def _check(c, keys, seed, what):
    for call in range(2):
        c.update(keys if call == 0 else keys[::-1].copy(), grads_for(seed, call * len(keys), len(keys), c.D))
    counts = np.bincount(keys.astype(np.int64))
    stats = c.ctx.batch_stats()
    assert stats["long_rows"] == int((counts > 1024).sum())
    assert stats["long_items"] == int(counts[counts > 1024].sum())
    log(what, len(keys), c.compare(what))
    if c.propagation == 0:
        c.check_invariant()


RULES = [(0, 0), (1, 0), (0, 1), (1, 1)]


@pytest.mark.parametrize("opt,comb", RULES)
@pytest.mark.parametrize("D,k,S", [(128, 4, 5), (36, 10, 11), (200, 2, 64), (16, 1, 2), (512, 3, 7)])
def test_runs_and_stripes_around_the_thresholds(D, k, S, opt, comb):
    rng = np.random.default_rng(11)
    R = k * 3000
    lens = [1, 2, 15, 16, 17, 47, 48, 49, 56, 57, 63, 64, 65, 127, 128, 129, 255, 511, 512, 513, 1023, 1024, 1025, 1500, 3000]
    stripes = rng.permutation(R // k)[:2 * len(lens)]
    keys = []
    for i, m in enumerate(lens):
        keys.append(np.full(m, stripes[2 * i] * k + i % k))                 # one entry has all of a stripe's updates
        keys.append(stripes[2 * i + 1] * k + rng.integers(0, k, m))         # ... or its entries share them
    keys.append(rng.integers(0, R, 6000))
    keys = rng.permutation(np.concatenate(keys)).astype(np.uint64)
    c = Case(R, D, k, S, max_batch=len(keys), seed=43, optimizer=opt, momentum=0.9, combine=comb)
    _check(c, keys, 43, f"thresholds {(D, k, S, opt, comb)}")


@pytest.mark.parametrize("prop", [0, 2])
@pytest.mark.parametrize("R,D,k,S,n", [
    (4 * 5000, 128, 4, 5, 2049), (4 * 5000, 128, 4, 5, 7 * 512 + 1), (4 * 5000, 128, 4, 5, 32 * 512 + 1), (4 * 100000, 8, 4, 5, (1 << 17) + 1),
    (4 * 60000, 8, 4, 5, 1 << 18), (4 * 60000, 4, 4, 5, (1 << 18) + 1), (2 * 60000, 12, 2, 3, (1 << 19) - 1),
    (2 * 60000, 12, 2, 3, 1 << 19), (2 * 60000, 12, 2, 3, (1 << 19) + 1), (4 * 31, 12, 4, 5, 1 << 18), (4 * 31, 12, 4, 5, (1 << 18) + 1),
    (4 * 32, 12, 4, 5, (1 << 18) + 1),
    (63 * 30, 1024, 63, 64, 5000), (7, 64, 7, 8, 4000), (1 << 20, 128, 4, 5, 33)])
def test_sizes_at_the_edges_of_the_plan(R, D, k, S, n, prop):
    c = Case(R, D, k, S, max_batch=n, seed=47, propagation=prop)
    _check(c, si.uniform_keys(47, 0, n, R), 47, f"plan {(R, D, k, S, n, prop)}")


@pytest.mark.parametrize("opt,comb", RULES)
@pytest.mark.parametrize("D,k,S", [(20, 4, 5), (12, 10, 11)])
def test_one_bucket_gets_everything(D, k, S, opt, comb):
    """Keys whose stripes all fall into one bucket of the plan: more stripes than the 640 that the LDS table of an oversized
    bucket may hold, so that it is worked off in parts, and more heavy ones than the 16 that a part may have, of 256 updates
    (the fewest) to more than a list takes; none of them hot in the sample."""
    n, stripes = 40000, 1 << 20
    g = np.arange(stripes, dtype=np.uint32)
    mine = g[bp.bucket_of(g, n) == 7]
    rng = np.random.default_rng(3)
    mine = rng.permutation(mine)
    assert len(mine) > 760
    limit = bp.heavy_stripe(k)
    heavy = [limit - 1, limit, limit + 1, 300, 511, 512, 513, bp.bucket_cap(), bp.bucket_cap() + 1, 2500] + [400] * 12
    light = mine[len(heavy):]
    sampled = bp.sample_positions(n)
    rest = rng.permutation(np.setdiff1d(np.arange(n), sampled))
    at = np.empty(n, np.int64)
    at[sampled] = light[np.arange(len(sampled)) % len(light)]                   # the sample sees light stripes, each once
    fill = np.repeat(mine[:len(heavy)], heavy)
    at[rest] = np.concatenate([fill, light[np.arange(len(rest) - len(fill)) % len(light)]])
    keys = at * k + rng.integers(0, k, n)
    assert len(np.unique(at)) > 640 and len(bp.hot_stripes(keys, k)) == 0
    c = Case(k * stripes, D, k, S, max_batch=n, seed=53, optimizer=opt, momentum=0.9, combine=comb)
    _check(c, keys.astype(np.uint64), 53, f"one bucket {(k, opt, comb)}")


def test_two_runs_are_bit_identical():
    n, R = 60000, 4 * 20000
    keys = si.zipf_keys(5, 0, n, 1 << 16, 1 << 16)
    outs = []
    for _ in range(2):
        c = Case(R, 128, 4, 5, n, seed=3)
        c.ctx.update(torch.from_numpy(keys.view(np.int64)).cuda(), grads_for(3, 0, n, 128))
        assert c.ctx.status() == 0
        outs.append([t.clone() for t in (c.E, c.A, c.PE, c.PA, c.ld, c.lp)])
    for x, y in zip(*outs):
        assert torch.equal(x, y)


@pytest.mark.parametrize("prop", [0, 2])
@pytest.mark.parametrize("opt,comb", RULES)
@pytest.mark.parametrize("R,D,k,S,n", [(4 * 900, 128, 4, 5, 30000), (10 * 3000, 68, 10, 13, 9001), (2 * 77, 256, 2, 64, 2000),
                                       (3 * 50, 300, 3, 5, 1 << 16)])
def test_same_as_the_general_path(R, D, k, S, n, opt, comb, prop):
    """The bucket path against the sort and the chain tiers (the knob sends a batch there): two fp64 chains in arrival
    order, each rounded once, so the tables agree but for re-association across a rounding boundary (~1e-6 of the
    elements, one ulp); the counters are equal."""
    keys = si.zipf_keys(59, 0, n, 1 << 14, 1 << 14) % np.uint64(R)
    kt, g = torch.from_numpy(keys.view(np.int64)).cuda(), grads_for(59, 0, n, D)
    out = []
    for general in (False, True):
        c = Case(R, D, k, S, max_batch=n, seed=59, optimizer=opt, momentum=0.9, combine=comb, propagation=prop)
        if general:
            c.ctx.tune(1, 0xFFFFFFFF)              # ECRM_TUNE_MID_MIN_ROWS: the chain tiers, no one-workgroup walk
        c.ctx.update(kt, g)
        assert c.ctx.status() == 0
        out.append((c.E, c.A, c.PE, c.PA, c.ld, c.lp))
    for a, b in zip(*out):
        if a.dtype == torch.float32:
            assert int((a != b).sum()) <= 1e-4 * a.numel() + 2
            assert torch.allclose(a, b, rtol=1e-5, atol=1e-9)
        else:
            assert torch.equal(a, b)


@pytest.mark.parametrize("opt,comb", RULES)
@pytest.mark.parametrize("R,D,n_stripes", [(10 * 64, 16, 40), (10 * 64, 132, 12)])
def test_heavy_stripes_of_many_entries(R, D, n_stripes, opt, comb):
    """Heavy stripes all of whose ten entries were hit, so that a workgroup exchanges sums for one entry right after the
    other: entries of one, two and three rounds of 1024 updates in changing order.  Against the oracle, and twice from
    the same start, which has to give the same bits."""
    k, S = 10, 11
    rng = np.random.default_rng(71)
    lens = [130, 1024, 200, 1025, 150, 2049, 131, 257, 2048, 300]
    keys = [np.full(lens[(j + 3 * s) % k], s * k + j) for s in range(n_stripes) for j in range(k)]
    keys = rng.permutation(np.concatenate(keys + [rng.integers(0, R, 999)])).astype(np.uint64)
    c = Case(R, D, k, S, max_batch=len(keys), seed=67, optimizer=opt, momentum=0.9, combine=comb)
    kt, g = torch.from_numpy(keys.view(np.int64)).cuda(), grads_for(67, 0, len(keys), D)
    tables = (c.E, c.A, c.PE, c.PA, c.ld, c.lp)
    start, runs = [t.clone() for t in tables], []
    for _ in range(2):
        for t, s in zip(tables, start):
            t.copy_(s)
        c.ctx.update(kt, g)
        runs.append([t.clone() for t in tables])
    for a, b in zip(*runs):
        assert torch.equal(a, b)
    c.oracle_update(keys, g)
    log("heavy stripes of many entries", (R, D, opt, comb), c.compare("heavy stripes of many entries"))


@pytest.mark.parametrize("opt,comb", RULES)
@pytest.mark.parametrize("n,D,k,S", [(8192, 36, 4, 5), (70001, 128, 10, 11), (200000, 12, 1, 2)])
def test_stripes_taken_for_hot_by_chance(n, D, k, S, opt, comb):
    """Stripes that fill just as many sampled positions as make them hot, and hold fewer, as many and more updates in all than
    the number below which they are given back to the ordinary buckets; one whose updates are all of one member."""
    rng = np.random.default_rng(n)
    R = k * (n // 8)
    at, hits = bp.sample_positions(n), int(bp.lib().plan_hot_hits(n))
    keys = rng.integers(k * 16, R, n)
    off = rng.permutation(np.setdiff1d(np.arange(n), at))
    at = rng.permutation(at)
    limit = max(bp.shared_stripe(n, k) // 2, bp.heavy_stripe(k))               # few of them are hot
    totals = [hits, hits + 1, 100, 128, 200, limit - 1, limit, limit + 1, limit + 50]
    for g, total in enumerate(totals):
        mine, at, off = np.concatenate([at[:hits], off[:total - hits]]), at[hits:], off[total - hits:]
        keys[mine] = g * k + (k - 1 if g % 3 == 2 else rng.integers(0, k, total))
    assert set(range(len(totals))) <= set(bp.hot_stripes(keys, k).tolist())
    assert (np.bincount(keys // k)[:len(totals)] == totals).all()
    c = Case(R, D, k, S, max_batch=n, seed=73, optimizer=opt, momentum=0.9, combine=comb)
    _check(c, keys.astype(np.uint64), 73, f"hot by chance {(n, opt, comb)}")


@pytest.mark.parametrize("opt,comb", RULES)
@pytest.mark.parametrize("D,k,S,n", [(128, 4, 5, 30000), (300, 2, 3, 60000), (36, 10, 11, 20000), (1024, 3, 5, 20000),
                                     (8, 63, 64, 40000), (64, 1, 2, 20000)])
@pytest.mark.parametrize("parity,many", [(True, True), (True, False), (False, True)])
def test_stripes_shared_by_a_workgroup(D, k, S, n, parity, many, opt, comb):
    """Stripes that do not end inside a window of 64 positions: around the window, around four updates to an entry from which
    they are shared, around the length from which they are not any more; spread evenly, with one run of half and of more
    than half of them, with an untouched entry, and with a run long enough to be heavy in a stripe that it dominates or not.
    In a batch of few and of many hot stripes, which decides what becomes of such a run."""
    rng = np.random.default_rng(D + k)
    limit, run = bp.shared_stripe(n, k), bp.heavy_run(n)
    sizes = [57, 58, 63, 64, 65, 71, 4 * k - 1, 4 * k, 4 * k + 1, 128, run, 2 * run - 1, 2 * run, 2 * run + 1, limit - 1, limit, limit + 1]
    stripes = rng.permutation(n // 8)[:4 * len(sizes)]
    keys = []
    for i, size in enumerate(sizes):
        even, half, more, most = (stripes[4 * i + j] * k for j in range(4))
        keys.append(even + np.arange(size) % k)
        keys.append(half + np.concatenate([np.full(size // 2, k - 1), rng.integers(0, k, size - size // 2)]))
        keys.append(more + np.concatenate([np.full(size // 2 + 1, 0), np.arange(size - size // 2 - 1) % k]))
        keys.append(most + np.concatenate([np.full(size - size // 8, k // 2), rng.integers(k // 2, k, size // 8)]))
    keys = np.concatenate(keys)
    assert len(keys) < n
    R, hits = k * (n // 8 + 40), int(bp.lib().plan_hot_hits(n))
    at = rng.permutation(bp.sample_positions(n))[:40 * hits if many else 0]      # 40 stripes behind the others' are hot
    rest = rng.permutation(np.setdiff1d(np.arange(n), at))
    batch = np.empty(n, np.int64)
    batch[at] = k * (n // 8 + np.arange(len(at)) % 40)
    batch[rest[:len(keys)]] = keys
    batch[rest[len(keys):]] = rng.integers(0, k * (n // 8), n - len(at) - len(keys))
    assert (len(bp.hot_stripes(batch, k)) > 32) == many
    keys = batch.astype(np.uint64)
    c = Case(R, D, k, S, max_batch=n, seed=79, optimizer=opt, momentum=0.9, combine=comb, propagation=0 if parity else 2)
    _check(c, keys, 79, f"shared {(D, k, n, parity, many, opt, comb)}")


@pytest.mark.parametrize("opt,comb", RULES)
@pytest.mark.parametrize("R,D,k,S,n,hot", [
    (4 * 64, 36, 4, 5, 8203, 1.0), (4 * 64, 36, 4, 5, 8204, 1.0), (4 * 64, 132, 4, 5, 10 * 1024 + 1, 1.0), (1, 16, 1, 2, 1 << 16, 1.0),
    (4 * 5000, 128, 4, 5, 70001, 0.5), (10 * 100, 20, 10, 11, 200003, 0.9), (63 * 3, 8, 63, 64, 50000, 0.0), (7 * 2, 1024, 7, 8, 30000, 1.0),
    (200, 4, 4, 5, 1 << 19, 0.6)])
def test_runs_cut_into_segments(R, D, k, S, n, hot, opt, comb):
    """One row with a share of the batch, few rows with all of it: around the stripe length from which runs are cut into
    segments, runs of whole segments and of one update more, entries without an update in such a stripe.  Against the
    oracle, and twice from the same start, which has to give the same bits."""
    rng = np.random.default_rng(n)
    keys = rng.integers(0, R, n)
    keys[rng.random(n) < hot] = R // 2
    keys[:3 * k] = np.concatenate([np.arange(k), np.full(2 * k, R - 1)])
    assert (np.bincount(keys // k).max() >= bp.split_stripe(n, D)) == (n != 8203)
    keys = rng.permutation(keys).astype(np.uint64)
    c = Case(R, D, k, S, max_batch=n, seed=97, optimizer=opt, momentum=0.9, combine=comb)
    kt, g = torch.from_numpy(keys.view(np.int64)).cuda(), grads_for(97, 0, n, D)
    tables = (c.E, c.A, c.PE, c.PA, c.ld, c.lp)
    start, runs = [t.clone() for t in tables], []
    for _ in range(3):
        for t, s in zip(tables, start):
            t.copy_(s)
        c.ctx.update(kt, g)
        runs.append([t.clone() for t in tables])
    for other in runs[1:]:
        for a, b in zip(runs[0], other):
            assert torch.equal(a, b)
    c.oracle_update(keys, g)
    counts = np.bincount(keys.astype(np.int64))
    stats = c.ctx.batch_stats()
    assert stats["long_rows"] == int((counts > 1024).sum()) and stats["long_items"] == int(counts[counts > 1024].sum())
    log("segments", (R, D, k, n, hot, opt, comb), c.compare("segments"))


def test_replay_through_the_sort_of_updates_held_back_by_the_buckets():
    """A recovery buffer of more than 2^19 updates: its replay goes through the sort, the updates before and after through
    buckets, on the same scratch buffer."""
    R, D, k, S, server, chunks, n, cap = 4 * 900, 20, 4, 5, 1, 3, 9000, (1 << 19) + 5
    c = Case(R, D, k, S, max_batch=cap, seed=101)
    c.ctx.fail_server(server)
    oracle.fail_server(c.hE, c.hA, c.hPE, c.hPA, k, S, server)
    bk, bg = torch.empty(2 * cap, dtype=torch.int64, device="cuda"), torch.empty(2 * cap, D, device="cuda")
    c.ctx.recovery_begin(server, chunks, bk, bg, cap)
    ses = RecoverySession(c.hE, c.hA, c.hPE, c.hPA, k, S, c.lr, c.eps, server, chunks, cap, c.hld, c.hlp, threads=8)
    first = 0

    def update():
        nonlocal first
        keys, g = si.zipf_keys(101, first, n, 1 << 14, 1 << 14) % np.uint64(R), grads_for(101, first, n, D)
        first += n
        c.ctx.update(torch.from_numpy(keys.view(np.int64)).cuda(), g)
        assert ses.update(keys, g.cpu().numpy())

    for _ in range(ses.chunks):
        update()
        c.ctx.recovery_lock()
        ses.lock()
        update()
        c.ctx.recovery_decode()
        ses.decode()
        assert c.ctx.recovery_state()["buffered"] == len(ses.buf_keys) > 0
        c.ctx.recovery_unlock()
        ses.unlock()
        update()
    assert not c.ctx.recovery_state()["active"]
    update()
    log("replay through the sort", c.compare("replay through the sort"))


@pytest.mark.parametrize("opt,comb", RULES)
def test_heavy_and_cut_up_stripes_inside_a_hip_graph(opt, comb):
    """Replays of a captured call with a run cut into segments, heavy stripes and shared ones, each against an eager call on a
    twin, with eager work and synchronisation in between: what a call's kernels count and hand on starts afresh."""
    R, D, k, S, n = 4 * 2000, 36, 4, 5, 30000
    rng = np.random.default_rng(109)
    keys = rng.integers(0, R, n)
    keys[::2] = 4321
    keys[1::16] = 999
    keys[3::32] = 1000 + rng.integers(0, 4, len(keys[3::32]))
    keys[5::150] = 2000 + rng.integers(0, 4, len(keys[5::150]))
    assert np.bincount(keys // k).max() >= bp.split_stripe(n, D)
    kt, g = torch.from_numpy(keys).cuda(), grads_for(109, 0, n, D)
    a, b = (Case(R, D, k, S, max_batch=n, seed=109, optimizer=opt, momentum=0.9, combine=comb) for _ in range(2))
    a.ctx.update(kt, g)
    b.ctx.update(kt, g)
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        a.ctx.update(kt, g, stream=side)
    for rep in range(4):
        graph.replay()
        b.ctx.update(kt, g)
        torch.cuda.synchronize()
        for x, y in zip((a.E, a.A, a.PE, a.PA, a.ld, a.lp), (b.E, b.A, b.PE, b.PA, b.ld, b.lp)):
            assert torch.equal(x, y), f"replay {rep}"
        (a.E.sum() + b.E.sum()).item()
    assert a.ctx.status() == 0
