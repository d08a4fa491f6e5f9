"""A scenario's result does not depend on how many waves its batch gives it:
batches that run unsplit, split in two and split as far as the shape allows
agree bit for bit, in each workgroup shape, and with the CPU oracle."""
import numpy as np
import pytest

from oracle import nr as onr
from tests.gpu_common import angle_err, to_dev
from workloads import transmission as tx

pytestmark = pytest.mark.gpu


# the largest grid of each shape and the smallest, with batches past each split's room
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,batches", [(64, (5,)), (65, (3, 1100, 2200)), (256, (3, 1100, 2200)), (257, (3, 300, 600)),
                                       (1024, (3, 300, 600)), (1025, (3, 300, 600)), (2048, (3, 300, 600)),
                                       (2049, (3, 300)), (4100, (2,))])
def test_split_changes_no_bit(n, batches, precision):
    import torch
    from paper_2605_14103_amd import pf
    cfg = tx.TxConfig(f"g{n}", n_bus=n, n_pv=max(1, round(0.15 * n)), n_branch=round(1.3 * n), batch=batches[-1],
                      seed=n, perturbation="uniform")
    grid = tx.make_grid(cfg)
    batch = tx.make_batch(grid, cfg)
    ctx = pf.Context(0)
    net = pf.TxNetwork.from_grid(ctx, grid)
    few = batches[0]
    got, grads = [], []
    for B in batches:
        p, q, vm = (to_dev(a[:B]) for a in (batch.p_inj, batch.q_inj, batch.vm_set))
        res = net.solve(p, q, vm, precision=pf.precision(precision))
        _, dl_dv = net.branch_loss(res.v)
        gp, gq, its, ok = net.adjoint(res.v, dl_dv)
        torch.cuda.synchronize()
        assert res.converged.cpu().numpy().all() and ok.cpu().numpy().all()
        got.append([x[:few].cpu().numpy() for x in (res.v, res.newton_iters, res.gmres_iters, res.mismatch)])
        grads.append([x[:few].cpu().numpy() for x in (gp, gq, its)])
    net.close()
    ctx.close()
    for other, g in zip(got[1:], grads[1:]):
        assert all(np.array_equal(x, y) for x, y in zip(got[0], other))
        assert all(np.array_equal(x, y) for x, y in zip(grads[0], g))
    V, _, ok, _ = onr.nr_solve_batch(grid, batch, columns=np.arange(few))
    assert ok.all()
    da, dm = angle_err(got[0][0], V)
    assert da <= 1e-6 and dm <= 1e-6   # the solver's tolerance of 1e-8 pu mismatch


# the direct step: unsplit only, and split in each shape with the schedule in LDS, the
# factor in LDS and the factor in device memory
@pytest.mark.parametrize("n,batches", [(3, (2,)), (64, (5, 600)), (65, (3, 1100)), (256, (3, 1100)), (257, (3, 600)),
                                       (700, (3, 300)), (1025, (3, 300)), (2048, (2, 300))])
def test_direct_split_changes_no_bit(n, batches):
    import torch
    from paper_2605_14103_amd import pf
    cfg = tx.TxConfig(f"d{n}", n_bus=n, n_pv=max(1, round(0.15 * n)), n_branch=max(n - 1, round(1.3 * n) - 1),
                      batch=batches[-1], seed=n, perturbation="uniform")
    grid = tx.make_grid(cfg)
    batch = tx.make_batch(grid, cfg)
    ctx = pf.Context(0)
    net = pf.TxNetwork.from_grid(ctx, grid)
    few = batches[0]
    got = []
    for B in batches:
        res = net.solve(*(to_dev(a[:B]) for a in (batch.p_inj, batch.q_inj, batch.vm_set)), nr_direct=1)
        torch.cuda.synchronize()
        assert res.converged.cpu().numpy().all()
        got.append([x[:few].cpu().numpy() for x in (res.v, res.newton_iters, res.mismatch)])
    net.close()
    ctx.close()
    for other in got[1:]:
        assert all(np.array_equal(x, y) for x, y in zip(got[0], other))
    V, it, ok, _ = onr.nr_solve_batch(grid, batch, columns=np.arange(few))
    assert ok.all() and np.array_equal(got[0][1], it)   # both take exact Newton steps
    da, dm = angle_err(got[0][0], V)
    assert da <= 1e-6 and dm <= 1e-6   # the solver's tolerance of 1e-8 pu mismatch


# a block-diagonal preconditioner takes cycles of up to thirty steps; unsplit, their dot
# products run over two vectors a round in each shape of four units
@pytest.mark.parametrize("n,batches", [(200, (3, 4200)), (300, (3, 1100)), (1500, (2, 600))])
def test_long_cycles_change_no_bit(n, batches):
    import torch
    from paper_2605_14103_amd import pf
    cfg = tx.TxConfig(f"b{n}", n_bus=n, n_pv=max(1, round(0.15 * n)), n_branch=round(1.3 * n), batch=batches[-1],
                      seed=n, perturbation="uniform")
    grid = tx.make_grid(cfg)
    batch = tx.make_batch(grid, cfg)
    ctx = pf.Context(0)
    net = pf.TxNetwork.from_grid(ctx, grid, precond_block=32)
    few = batches[0]
    got = []
    for B in batches:
        res = net.solve(*(to_dev(a[:B]) for a in (batch.p_inj, batch.q_inj, batch.vm_set)))
        _, dl_dv = net.branch_loss(res.v)
        gp, gq, its, _ = net.adjoint(res.v, dl_dv)
        torch.cuda.synchronize()
        got.append([x[:few].cpu().numpy() for x in (res.v, res.newton_iters, res.gmres_iters, res.mismatch,
                                                    res.converged, gp, gq, its)])
    net.close()
    ctx.close()
    assert all(np.array_equal(x, y) for x, y in zip(*got))
    assert (got[0][2] > 10 * got[0][1]).any()   # cycles of many steps were run
    V, _, ok, _ = onr.nr_solve_batch(grid, batch, columns=np.arange(few))
    assert ok.all() and got[0][4].all()
    da, dm = angle_err(got[0][0], V)
    assert da <= 1e-6 and dm <= 1e-6   # the solver's tolerance of 1e-8 pu mismatch
