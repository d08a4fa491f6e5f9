"""The direct Newton step where a grid's factor just fits a CU's LDS: the
unsplit workgroup's bytes lie within 160 KB, those of a split one (it holds the
partial sums of more waves) past it.  Such grids solve at every batch size, and
a scenario's result does not depend on it."""
import numpy as np
import pytest

from oracle import nr as onr
from tests.gpu_common import angle_err, to_dev
from workloads import transmission as tx

pytestmark = pytest.mark.gpu


# 163752, 163656 and 163688 bytes unsplit (of 163840); 192 more split in four
@pytest.mark.parametrize("n,seed", [(901, 901), (900, 8), (900, 18)])
def test_factor_that_just_fits(n, seed):
    import torch
    from paper_2605_14103_amd import pf
    cfg = tx.TxConfig(f"g{n}", n_bus=n, n_pv=round(0.15 * n), n_branch=round(1.3 * n), batch=300, seed=seed,
                      perturbation="uniform")
    grid = tx.make_grid(cfg)
    batch = tx.make_batch(grid, cfg)
    ctx = pf.Context(0)
    net = pf.TxNetwork.from_grid(ctx, grid)
    got = []
    for B in (2, 300):
        res = net.solve(*(to_dev(a[:B]) for a in (batch.p_inj, batch.q_inj, batch.vm_set)), nr_direct=1)
        torch.cuda.synchronize()
        assert res.converged.cpu().numpy().all()
        got.append([x[:2].cpu().numpy() for x in (res.v, res.newton_iters, res.mismatch)])
    net.close()
    ctx.close()
    assert all(np.array_equal(x, y) for x, y in zip(*got))
    V, it, ok, _ = onr.nr_solve_batch(grid, batch, columns=np.arange(2))
    assert ok.all() and np.array_equal(got[0][1], it)   # both take exact Newton steps
    da, dm = angle_err(got[0][0], V)
    assert da <= 1e-6 and dm <= 1e-6   # the solver's tolerance of 1e-8 pu mismatch
