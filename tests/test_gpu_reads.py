"""Reads where the flat copy and the shared answers can go wrong: rows of any width beside the 16 bytes a lane moves, stripes of
one member and of many, numbers of requests around what a wave takes (4 to 64), more requests than the scratch buffer serves at a
time, or a launch takes, buffers around the largest whose waiting updates are sorted in two launches to a digit, and waiting runs on either side of what one wave walks (128) and of a workgroup's round (1024), requested many times."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
import synth_inputs as si
from ecrm_case import Case, grads_for
from oracle.recovery_session import RecoverySession

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,k,S", [(4, 1, 2), (12, 3, 4), (60, 5, 7), (128, 4, 5), (260, 10, 11), (1024, 2, 5)])
def test_degraded_read_widths(D, k, S):
    R, n = k * 500, 3001 if D > 12 else 1100003          # the latter: 64 requests to a wave
    c = Case(R, D, k, S, max_batch=64, seed=31)
    lost = S - 1
    c.ctx.fail_server(lost)
    oracle.fail_server(c.hE, c.hA, c.hPE, c.hPA, k, S, lost)
    keys = si.uniform_keys(32, 0, n, R)
    he, ha = oracle.degraded_read(c.hE, c.hA, c.hPE, c.hPA, k, S, keys, lost)
    kt = torch.from_numpy(keys.view(np.int64)).cuda()
    for m in (1, 3, 5, 63, 64, 65, n):
        oe, oa = torch.full((m + 1, D), -7.0, device="cuda"), torch.full((m + 1, D), -7.0, device="cuda")
        c.ctx.degraded_read(kt[:m], lost, oe, oa)
        np.testing.assert_array_equal(oe[:m].cpu().numpy(), he[:m])
        np.testing.assert_array_equal(oa[:m].cpu().numpy(), ha[:m])
        assert bool((oe[m] == -7.0).all()) and bool((oa[m] == -7.0).all())
    assert c.ctx.status() == 0


@pytest.mark.parametrize("D,k,S,server,opt", [(4, 3, 5, 1, 0), (128, 4, 5, 2, 0), (36, 2, 3, 0, 1), (264, 10, 11, 7, 0)])
@pytest.mark.parametrize("locked", [False, True])
def test_shared_answers(D, k, S, server, opt, locked):
    R, cap = k * 600, 9000
    rng = np.random.default_rng(D)
    c = Case(R, D, k, S, max_batch=cap, seed=33, optimizer=opt, momentum=0.9)
    _, _, ds, _ = oracle.route(np.arange(R, dtype=np.uint64), R, k, S)
    rows = np.nonzero(ds == server)[0]
    lens = [126, 127, 128, 129, 1023, 1024, 1025, 2049, 1, 2]
    rows = rng.permutation(rows[rows < R // 2])[:len(lens)]        # of the first chunk
    keys = rng.permutation(np.concatenate([np.repeat(rows, lens), rng.integers(0, R, 800)])).astype(np.uint64)
    c.ctx.fail_server(server)
    oracle.fail_server(c.hE, c.hA, c.hPE, c.hPA, k, S, server)
    bk, bg = torch.empty(2 * cap, dtype=torch.int64, device="cuda"), torch.empty(2 * cap, D, device="cuda")
    c.ctx.recovery_begin(server, 2, bk, bg, cap)
    ses = RecoverySession(c.hE, c.hA, c.hPE, c.hPA, k, S, c.lr, c.eps, server, 2, cap, c.hld, c.hlp, optimizer=opt,
                          momentum=0.9, combine=0, threads=4)
    if locked:                                            # more waits, stored entries among it
        c.ctx.recovery_lock()
        ses.lock()
    g = grads_for(33, 0, len(keys), D)
    c.ctx.update(torch.from_numpy(keys.view(np.int64)).cuda(), g)
    assert ses.update(keys, g.cpu().numpy())
    # every entry many times, hot ones more often; more requests than max_batch: three parts
    some = np.concatenate([np.arange(R), np.repeat(rows, 300)])
    sample = rng.choice(some, 2 * cap + 77).astype(np.uint64)
    want_e, want_a = ses.read(np.arange(R, dtype=np.uint64))
    st = torch.from_numpy(sample.view(np.int64)).cuda()
    oe, oa = torch.empty(len(sample), D, device="cuda"), torch.empty(len(sample), D, device="cuda")
    for _ in range(2):
        oe.fill_(float("nan"))
        oa.fill_(float("nan"))
        c.ctx.recovery_read(st, oe, oa)
        assert c.ctx.status() == 0
        np.testing.assert_allclose(oe.cpu().numpy(), want_e[sample], rtol=1e-5, atol=5e-7)
        np.testing.assert_allclose(oa.cpu().numpy(), want_a[sample], rtol=1e-5, atol=1e-9)
    only = torch.empty_like(oe)
    c.ctx.recovery_read(st, only)
    assert torch.equal(only, oe)
    first = {}
    for i, x in enumerate(sample.tolist()):               # requests for one entry get one answer
        first.setdefault(x, i)
    assert torch.equal(oe, oe[torch.tensor([first[x] for x in sample.tolist()], device="cuda")])


def _hip():
    """The HIP runtime this process has loaded."""
    with open("/proc/self/maps") as f:
        return C.CDLL(next(line.split()[-1] for line in f if "libamdhip64" in line))


def _launches(call):
    """How many launches a call enqueues, counted in a graph captured of it (which is not run)."""
    hip, stream = _hip(), torch.cuda.Stream()
    torch.cuda.synchronize()
    handle, graph, nodes = C.c_void_p(stream.cuda_stream), C.c_void_p(), C.c_size_t(0)
    assert hip.hipStreamBeginCapture(handle, 1) == 0         # only what this thread does
    try:
        call(stream)
    finally:
        assert hip.hipStreamEndCapture(handle, C.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, C.byref(nodes)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return nodes.value


def _waiting(R, D, k, S, server, cap, max_batch, keys, seed=35):
    """A recovery with the updates of `keys` to lost entries and to the first half of the stripes waiting."""
    c = Case(R, D, k, S, max_batch=max_batch, seed=seed)
    bk, bg = torch.empty(2 * cap, dtype=torch.int64, device="cuda"), torch.empty(2 * cap, D, device="cuda")
    c.ctx.recovery_begin(server, 2, bk, bg, cap)
    ses = RecoverySession(c.hE, c.hA, c.hPE, c.hPA, k, S, c.lr, c.eps, server, 2, cap, c.hld, c.hlp, threads=4)
    c.ctx.recovery_lock()
    ses.lock()
    for at in range(0, len(keys), max_batch):
        part = keys[at:at + max_batch]
        g = grads_for(seed, at, len(part), D)
        c.ctx.update(torch.from_numpy(part.view(np.int64)).cuda(), g)
        assert ses.update(part, g.cpu().numpy())
    return c, ses


def test_a_read_of_many_requests_is_as_many_launches():
    """A context made for small batches reads as many entries as it likes: the launches do not follow the requests."""
    R, D, k, S, cap = 4 * 500, 16, 4, 5, 256
    keys = np.random.default_rng(2).integers(0, R, cap).astype(np.uint64)
    c, ses = _waiting(R, D, k, S, 1, cap, cap, keys)
    count = []
    for n in (cap, 8 * cap, 100 * cap + 1):
        sample = np.random.default_rng(n).integers(0, R, n).astype(np.uint64)
        st, oe = torch.from_numpy(sample.view(np.int64)).cuda(), torch.full((n + 1, D), -7.0, device="cuda")
        c.ctx.recovery_read(st, oe[:n])
        want, _ = ses.read(sample)
        np.testing.assert_allclose(oe[:n].cpu().numpy(), want, rtol=1e-5, atol=5e-7)
        assert bool((oe[n] == -7.0).all())
        count.append(_launches(lambda s: c.ctx.recovery_read(st, oe[:n], stream=s)))
    assert count[0] == count[1] == count[2] <= 8


@pytest.mark.parametrize("cap", [1, 127, 128, 1024, 1025, 40000, 1 << 18, (1 << 18) + 1])
@pytest.mark.parametrize("R", [4 * 60, 4 * 3000, 4 * 70000])        # one, two and three digits
def test_waiting_lists(cap, R):
    D, k, S = 8, 4, 5
    rng = np.random.default_rng(cap + R)
    m = min(cap, 30000)
    keys = rng.integers(0, R, m)
    keys[::3] = rng.integers(0, min(R, 40), len(keys[::3]))           # entries with many among them
    c, ses = _waiting(R, D, k, S, 2, cap, max(cap, 64), keys.astype(np.uint64))
    sample = np.concatenate([rng.choice(keys, 3000), rng.integers(0, R, 3000)]).astype(np.uint64)
    want_e, want_a = ses.read(sample)
    st = torch.from_numpy(sample.view(np.int64)).cuda()
    for n in (len(sample), min(cap, 64)):                             # more than the scratch buffer serves, and fewer
        oe, oa = torch.full((n, D), float("nan"), device="cuda"), torch.full((n, D), float("nan"), device="cuda")
        for _ in range(2):
            c.ctx.recovery_read(st[:n], oe, oa)
        np.testing.assert_allclose(oe.cpu().numpy(), want_e[:n], rtol=1e-5, atol=5e-7)
        np.testing.assert_allclose(oa.cpu().numpy(), want_a[:n], rtol=1e-5, atol=1e-9)
    assert c.ctx.status() == 0


def test_more_requests_than_a_launch_takes():
    """2^32 requests and a few: with as many threads in one launch as requests, it was refused."""
    n, R, D, k, S, cap = (1 << 32) + 77, 4 * 250, 4, 4, 5, 300
    if torch.cuda.mem_get_info()[0] < n * (8 + 4 * D) + (8 << 30):
        pytest.skip("not enough memory on the device")
    c, ses = _waiting(R, D, k, S, 3, cap, cap, np.random.default_rng(4).integers(0, R, cap).astype(np.uint64))
    keys, out = torch.empty(n, dtype=torch.int64, device="cuda"), torch.empty(n, D, device="cuda")
    tables = torch.arange(R, device="cuda").repeat(1 << 18)          # whole tables, a part of the requests that torch handles
    parts = range(0, n, len(tables))
    for at in parts:
        keys[at:at + len(tables)] = tables[:min(len(tables), n - at)]
    want_waiting, _ = ses.read(np.arange(R, dtype=np.uint64))
    lost = oracle.degraded_read(c.hE, c.hA, c.hPE, c.hPA, k, S, np.arange(R, dtype=np.uint64), 3)[0]
    for read, want, atol in ((lambda: c.ctx.degraded_read(keys, 3, out), lost, 5e-7),
                             (lambda: c.ctx.recovery_read(keys, out), want_waiting, 5e-7)):
        for at in parts:
            out[at:at + len(tables)] = float("nan")
        read()
        assert c.ctx.status() == 0
        whole = torch.from_numpy(want).cuda()
        for at in parts:
            rows = out[at:at + len(tables)]
            full = len(rows) // R * R
            assert full == 0 or float((rows[:full].view(-1, R, D) - whole).abs().max()) <= atol
            assert full == len(rows) or float((rows[full:] - whole[:len(rows) - full]).abs().max()) <= atol
    del keys, out
    torch.cuda.empty_cache()
