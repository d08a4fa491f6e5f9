"""Branch loss and its gradient at the edges of the workgroup sizes that the
number of buses picks, against the oracle."""
import numpy as np
import pytest

from oracle import adjoint as oadj
from tests.gpu_common import to_dev
from workloads import transmission as tx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 256, 257, 768, 769, 2100])
def test_branch_loss_sizes(n):
    from paper_2605_14103_amd import pf
    if n == 2:
        grid, _ = tx.two_bus(0.01, 0.05, 0.1, 0.03)
    else:
        grid = tx.make_grid(tx.TxConfig(f"g{n}", n_bus=n, n_pv=round(0.15 * n), n_branch=round(1.3 * n), batch=1,
                                        seed=n, perturbation="uniform"))
    rng = np.random.default_rng(n)
    V = 1 + 0.02 * (rng.standard_normal((3, n)) + 1j * rng.standard_normal((3, n)))
    ctx = pf.Context(0)
    net = pf.TxNetwork.from_grid(ctx, grid)
    loss, g = net.branch_loss(to_dev(V))
    only, none = net.branch_loss(to_dev(V), grad=False)
    loss, g, only = loss.cpu().numpy(), g.cpu().numpy(), only.cpu().numpy()
    net.close()
    ctx.close()
    assert none is None and np.array_equal(only, loss)
    # branch currents of order 1 from differences of admittances up to 50: 2e-14 each, and a sum of squares
    np.testing.assert_allclose(loss, oadj.branch_loss(grid, V.T), rtol=1e-11)
    # 2 sum |y| dI over a bus's branches (under forty of them)
    np.testing.assert_allclose(g, np.conj(oadj.branch_loss_grad(grid, V.T)).T, rtol=0, atol=1e-10)
