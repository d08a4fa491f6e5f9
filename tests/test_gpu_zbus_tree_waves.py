"""The tree form of the feeder solve in every workgroup size it is built for: the
fewest and the most buses of each, in one launch and in an engine's steps."""
import numpy as np
import pytest

from oracle import zbus as ozb
from tests.gpu_common import to_dev
from tests.test_gpu_zbus_tree import ATOL, _batch, _feeder

pytestmark = pytest.mark.gpu

WAVES = [1, 2, 3, 4, 5, 6, 8, 10, 13, 16]
BUSES = [nb for low, high in zip([0] + WAVES, WAVES) for nb in (64 * low + 1, 64 * high)]   # below the slack


@pytest.mark.parametrize("nb", BUSES)
def test_every_wave_count(nb):
    import torch
    from paper_2605_14103_amd import pf
    n = nb + 1
    fd = _feeder(n, "random")
    batch = _batch(fd, 4)
    ctx = pf.Context(0)
    net = pf.DistNetwork(ctx, n, fd.seg_from, fd.seg_to, fd.z_seg, [0, 1, 2], fd.v_slack, fd.wye_nodes,
                         fd.delta_nodes)
    assert n < 100 or ctx.bytes() < 16 * (3 * n) ** 2   # the tree form holds no dense Z
    res = net.solve(to_dev(batch.s_wye), to_dev(batch.s_delta), tol=1e-11)
    torch.cuda.synchronize()
    v, its, ok = res.v.cpu().numpy(), res.iters.cpu().numpy(), res.converged.cpu().numpy()
    # in steps: two scenarios from the start, two more an iteration later, in slots out of order
    eng = pf.Engine(net, hbm_bytes=64 << 20, n_streams=0, tol=1e-11)
    where, got, steps = {}, {}, 0
    stream = torch.cuda.current_stream()
    while len(got) < 4:
        if steps in (0, 1):
            ks, sl = ([0, 1], [5, 2]) if steps == 0 else ([2, 3], [0, 7])
            eng.admit(sl, batch.s_wye[ks], batch.s_delta[ks], stream=stream)
            where.update(zip(sl, ks))
        done, _ = eng.step(1, stream=stream)
        steps += 1
        assert steps < 100
        if done:
            r = eng.harvest(done, stream=stream)
            for j, s in enumerate(done):
                got[where[s]] = (r.v[j], r.iters[j], r.converged[j], r.mismatch[j])
    mis = res.mismatch.cpu().numpy()
    eng.close()
    net.close()
    ctx.close()
    assert ok.all() and mis.max() <= 1e-11
    for k in range(4):
        assert np.array_equal(got[k][0], v[k]) and got[k][1] == its[k] and got[k][2] and got[k][3] == mis[k]
    ref = ozb.zbus_solve(fd, batch)
    assert ref.converged.all()
    np.testing.assert_allclose(v, ref.v, rtol=0, atol=ATOL)
