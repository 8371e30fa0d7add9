"""The one-launch append and replay of held-back updates where its tiles can go wrong: batches around one tile and around the
sizes at which a thread takes one, two and four updates, a buffer that is exactly full, one update too small, or far larger
than what waits in it, and slots that are used again."""
import numpy as np
import pytest
import torch

import oracle
from ecrm_case import Case, grads_for
from oracle.recovery_session import RecoverySession

pytestmark = pytest.mark.gpu


def _start(n, R, D, k, S, server, cap, opt=0):
    c = Case(R, D, k, S, max_batch=max(n, cap), seed=71, optimizer=opt, momentum=0.9)
    c.ctx.fail_server(server)
    oracle.fail_server(c.hE, c.hA, c.hPE, c.hPA, k, S, server)
    c.bk = torch.empty(2 * cap, dtype=torch.int64, device="cuda")
    c.bg = torch.empty(2 * cap, D, device="cuda")
    c.ctx.recovery_begin(server, 2, c.bk, c.bg, cap)
    ses = RecoverySession(c.hE, c.hA, c.hPE, c.hPA, k, S, c.lr, c.eps, server, 2, cap, c.hld, c.hlp, optimizer=opt,
                          momentum=0.9, combine=0, threads=8)
    return c, ses


def _both(c, ses, keys, g):
    c.ctx.update(torch.from_numpy(keys.view(np.int64)).cuda(), g)
    return ses.update(keys, g.cpu().numpy())


@pytest.mark.parametrize("n,cap", [(1, 1), (511, 512), (512, 2048), (513, 6000), (131072, 131072), (131073, 262144),
                                   (262145, 500000)])
def test_tiles(n, cap):
    R, D, k, S, server = 4 * 5000, 8 if n > 1000 else 132, 4, 5, 1
    c, ses = _start(n, R, D, k, S, server, cap)
    rng = np.random.default_rng(n)
    first = 0
    for chunk in range(2):
        for stage in ("before", "locked"):
            if stage == "locked":
                c.ctx.recovery_lock()
                ses.lock()
            keys = rng.integers(0, R, n).astype(np.uint64)
            assert _both(c, ses, keys, grads_for(71, first, n, D))
            first += n
            assert c.ctx.recovery_state()["buffered"] == len(ses.buf_keys)
        c.ctx.recovery_decode()
        ses.decode()
        c.ctx.recovery_unlock()
        ses.unlock()
        assert c.ctx.recovery_state()["buffered"] == len(ses.buf_keys)
    assert c.ctx.status() == 0 and not c.ctx.recovery_state()["active"]
    c.compare("hold tiles")


@pytest.mark.parametrize("n", [700, 140000])
def test_full_buffer(n):
    R, D, k, S, server = 4 * 5000, 8, 4, 5, 2
    rng = np.random.default_rng(3)
    keys = rng.integers(0, R, n).astype(np.uint64)
    probe = Case(R, D, k, S, max_batch=8, seed=71)
    held = int(RecoverySession(probe.hE, probe.hA, probe.hPE, probe.hPA, k, S, 0.01, 1e-8, server, 2, n).held(keys).sum())
    for cap, fits in ((held, True), (held - 1, False)):
        c, ses = _start(n, R, D, k, S, server, cap)
        before = [t.clone() for t in (c.E, c.A, c.PE, c.PA)]
        assert _both(c, ses, keys, grads_for(71, 0, n, D)) == fits
        assert c.ctx.status() == (0 if fits else -7)
        assert c.ctx.recovery_state()["buffered"] == (held if fits else 0)
        if not fits:                                     # rejected as a whole; the next one is not
            for t, b in zip((c.E, c.A, c.PE, c.PA), before):
                assert torch.equal(t.view(torch.int32), b.view(torch.int32))
            c.ctx.clear_status()
            bad = keys.copy()
            bad[n // 2] = R                              # out of range: nothing is applied, nothing appended
            c.ctx.update(torch.from_numpy(bad.view(np.int64)).cuda(), grads_for(71, 0, n, D))
            assert c.ctx.status() == -5 and c.ctx.recovery_state()["buffered"] == 0
            c.ctx.clear_status()
            assert _both(c, ses, keys[:n // 2], grads_for(71, 0, n // 2, D))
        c.ctx.recovery_lock(); ses.lock()
        c.ctx.recovery_decode(); ses.decode()
        c.ctx.recovery_unlock(); ses.unlock()
        assert c.ctx.recovery_state()["buffered"] == len(ses.buf_keys)
        more = rng.integers(0, R, min(n, cap) // 8).astype(np.uint64)        # takes the released slots
        assert _both(c, ses, more, grads_for(72, 0, len(more), D))
        c.ctx.recovery_lock(); ses.lock()
        c.ctx.recovery_decode(); ses.decode()
        c.ctx.recovery_unlock(); ses.unlock()
        assert c.ctx.status() == 0
        c.compare("full buffer")
