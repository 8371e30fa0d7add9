"""recovery_read where its walk of the waiting updates can go wrong: runs around the 64 places it looks at together and the
16 gradients it has in flight, the first and the last waiting entry, entries beside them with none, one waiting update in
all, repeated requests, without accumulators.  Against the protocol oracle, with the tolerance of a chain that the
library sums in one piece (rounded once on both sides)."""
import numpy as np
import pytest
import torch

import oracle
from ecrm_case import Case, grads_for
from oracle.recovery_session import RecoverySession

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens", [[1], [64], [1, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 500]])
@pytest.mark.parametrize("R,D,k,S,server,opt", [(4 * 3000, 128, 4, 5, 2, 0), (10 * 400, 200, 10, 11, 7, 1)])
def test_runs_of_waiting_updates(R, D, k, S, server, opt, lens):
    rng = np.random.default_rng(len(lens))
    c = Case(R, D, k, S, max_batch=8000, seed=61, optimizer=opt, momentum=0.9)
    _, _, ds, _ = oracle.route(np.arange(R, dtype=np.uint64), R, k, S)
    lost = np.nonzero(ds == server)[0]
    rows = np.concatenate([lost[:1], rng.permutation(lost[1:-1])[:max(len(lens) - 2, 0)], lost[-1:]])[:len(lens)]
    keys = np.concatenate([np.repeat(rows, lens), rng.choice(np.nonzero(ds != server)[0], 300)])
    keys = rng.permutation(keys).astype(np.uint64)
    c.ctx.fail_server(server)
    oracle.fail_server(c.hE, c.hA, c.hPE, c.hPA, k, S, server)
    bk = torch.empty(2 * 8000, dtype=torch.int64, device="cuda")
    bg = torch.empty(2 * 8000, D, device="cuda")
    c.ctx.recovery_begin(server, 1, bk, bg, 8000)
    ses = RecoverySession(c.hE, c.hA, c.hPE, c.hPA, k, S, c.lr, c.eps, server, 1, 8000, c.hld, c.hlp, optimizer=opt,
                          momentum=0.9, combine=0, threads=4)
    g = grads_for(61, 0, len(keys), D)
    c.ctx.update(torch.from_numpy(keys.view(np.int64)).cuda(), g)
    assert ses.update(keys, g.cpu().numpy())
    assert c.ctx.recovery_state()["buffered"] == len(ses.buf_keys) == sum(lens)
    sample = np.concatenate([rows, rows, lost[:3], lost[-3:], np.arange(50), [R - 1]]).astype(np.uint64)
    st = torch.from_numpy(sample.view(np.int64)).cuda()
    oe, oa = torch.empty(len(sample), D, device="cuda"), torch.empty(len(sample), D, device="cuda")
    c.ctx.recovery_read(st, oe, oa)
    assert c.ctx.status() == 0
    hE, hA = ses.read(sample)
    np.testing.assert_allclose(oe.cpu().numpy(), hE, rtol=1e-5, atol=5e-7)
    np.testing.assert_allclose(oa.cpu().numpy(), hA, rtol=1e-5, atol=1e-9)
    only = torch.empty_like(oe)
    c.ctx.recovery_read(st, only)
    assert torch.equal(only, oe)
