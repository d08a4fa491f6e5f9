"""The dense core's right-hand side where it has LDS of its own (short restarts
leave too few partial sums to share), its zeros over the norm's partial sums."""
import numpy as np
import pytest

from oracle import nr as onr
from tests.gpu_common import angle_err, to_dev
from workloads import transmission as tx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,rtol", [("fp64", 1e-7), ("fp64", 1e-3), ("mixed", 1e-3)])
@pytest.mark.parametrize("restart", [2, 5])
def test_core_beside_the_norm(precision, rtol, restart):
    import torch
    from paper_2605_14103_amd import pf
    cfg = tx.TX2000
    grid = tx.make_grid(cfg)
    batch = tx.make_batch(grid, cfg, batch=600)
    ctx = pf.Context(0)
    net = pf.TxNetwork.from_grid(ctx, grid)
    assert max(net.info["core_bp"], net.info["core_bpp"]) * 8 > 2 * (restart + 2) * 4 * 8
    opts = dict(gmres_restart=restart, gmres_max_restarts=100)
    got = []
    for B in (3, 300, 600):   # split in four, in two, unsplit
        res = net.solve(*(to_dev(a[:B]) for a in (batch.p_inj, batch.q_inj, batch.vm_set)), gmres_rtol=rtol,
                        forcing=0, precision=pf.precision(precision), **opts)
        _, dl_dv = net.branch_loss(res.v)
        gp, gq, its, ok = net.adjoint(res.v, dl_dv, **opts)
        torch.cuda.synchronize()
        assert res.converged.cpu().numpy().all() and ok.cpu().numpy().all()
        got.append([x[:3].cpu().numpy() for x in (res.v, res.newton_iters, res.gmres_iters, gp, gq, its)])
    net.close()
    ctx.close()
    for other in got[1:]:
        assert all(np.array_equal(x, y) for x, y in zip(got[0], other))
    V, _, ok, _ = onr.nr_solve_batch(grid, batch, columns=np.arange(3))
    da, dm = angle_err(got[0][0], V)
    assert ok.all() and da <= 1e-6 and dm <= 1e-6   # the solver's tolerance of 1e-8 pu mismatch
