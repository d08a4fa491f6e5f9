"""Device memory that a registered grid holds, with and without the direct
step's tables: a context whose budget was enough for it stays enough."""
import pytest

from tests.gpu_common import say, to_dev
from workloads import transmission as tx

pytestmark = pytest.mark.gpu


# (buses, bytes after registration, bytes after a direct solve of one scenario), as held before the
# preconditioner's first pass was laid out once per precision
@pytest.mark.parametrize("n,registered,direct", [
    (30, 90852, 116232), (64, 108284, 156376), (65, 243216, 314884), (256, 323524, 568188), (300, 864940, 1250536),
    (901, 1344424, 3482056), (2000, 2708332, 17724344)])
def test_grid_fits_its_budget(n, registered, direct):
    import torch
    from paper_2605_14103_amd import pf
    cfg = tx.TxConfig(f"g{n}", n_bus=n, n_pv=max(1, round(0.15 * n)), n_branch=round(1.3 * n), batch=1, seed=n,
                      perturbation="uniform")
    grid = tx.make_grid(cfg)
    batch = tx.make_batch(grid, cfg)
    for budget, solve in ((registered, False), (direct, True)):
        ctx = pf.Context(0, hbm_budget_bytes=budget)
        net = pf.TxNetwork.from_grid(ctx, grid)
        if solve:
            res = net.solve(*(to_dev(a) for a in (batch.p_inj, batch.q_inj, batch.vm_set)), nr_direct=1)
            torch.cuda.synchronize()
            assert res.converged.cpu().numpy().all()
        say(f"{n} buses hold {ctx.bytes()} of {budget} bytes")
        net.close()
        ctx.close()
