"""The general forms of the feeder solve (dense product and sparse factor), on
feeders with one closed loop, which the tree form does not take: row and column
tiles, the residual's slot templates, device-side exits, iteration caps, isolation of
bad scenarios and the serving engine's steps, against the CPU oracle."""
import numpy as np
import pytest

from oracle import zbus as ozb
from tests.gpu_common import HV_FLOOR_FEEDER, angle_err, assert_high_voltage, say, spread_cols, to_dev
from tests.test_gpu_serve import _collect
from workloads import feeder as fdm

pytestmark = pytest.mark.gpu

UPDATES = [(p, s) for p in ("fp64", "mixed") for s in (0, 1)]


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2605_14103_amd import pf
    assert torch.cuda.is_available()
    c = pf.Context(0)
    yield c
    c.close()


def _looped(cfg):
    return fdm.with_loop(fdm.make_feeder(cfg))


def _register(ctx, fd):
    """The feeder's network; asserts that it holds the general forms' dense Z."""
    from paper_2605_14103_amd import pf
    before = ctx.bytes()
    net = pf.DistNetwork.from_feeder(ctx, fd)
    n_free = fd.n_node - 3
    assert ctx.bytes() - before >= 12 * (2 * n_free) ** 2
    return net


def _solve(net, batch, **opts):
    import torch
    res = net.solve(to_dev(batch.s_wye), to_dev(batch.s_delta), **opts)
    torch.cuda.synchronize()
    return res


def _check(fd, batch, res, cols, label, setup=None):
    ref = ozb.zbus_solve(fd, fdm.FeederBatch(batch.s_wye[cols], batch.s_delta[cols]), setup=setup)
    assert ref.converged.all()
    da, dm = angle_err(res.v.cpu().numpy()[cols], ref.v)
    mis = res.mismatch.cpu().numpy()
    say(f"{label}: max angle err {da:.2e}, max |v| err {dm:.2e}, mismatch max {mis.max():.2e}")
    assert res.converged.cpu().numpy().all() and mis.max() <= 1e-8
    assert da <= 1e-6 and dm <= 1e-6


@pytest.mark.parametrize("precision,sparse", UPDATES)
def test_small_feeder_full(ctx, precision, sparse):
    """40 buses, 200 scenarios (two GEMM row tiles, ragged), all against the oracle."""
    from paper_2605_14103_amd import pf
    cfg = fdm.FeederConfig("feeder40", n_bus=40, max_depth=25, batch=200, seed=41)
    fd = _looped(cfg)
    batch = fdm.make_batch(fd, cfg)
    net = _register(ctx, fd)
    res = _solve(net, batch, precision=pf.precision(precision), zbus_sparse=sparse)
    _check(fd, batch, res, np.arange(200), f"loop40 {precision} sparse={sparse}")
    net.close()


def test_feeder300_full_batch_sampled(ctx):
    """300 buses, 4096 scenarios, each update in each precision."""
    from paper_2605_14103_amd import pf
    cfg = fdm.FEEDER300
    fd = _looped(cfg)
    batch = fdm.make_batch(fd, cfg)
    net = _register(ctx, fd)
    setup = ozb.zbus(fd)
    for precision, sparse in UPDATES:
        res = _solve(net, batch, precision=pf.precision(precision), zbus_sparse=sparse)
        assert_high_voltage(res.v.cpu().numpy(), HV_FLOOR_FEEDER, f"loop300 {precision} sparse={sparse}")
        _check(fd, batch, res, spread_cols(batch.batch, 32), f"loop300 {precision} sparse={sparse}", setup)
    net.close()


# 2097 and 2721 free nodes: nine and eleven slots of the residual (its template of sixteen), 33 and 43 column
# tiles of the GEMM with a ragged last one, levels of a large sparse factor
@pytest.mark.parametrize("n", [700, 908])
def test_large_feeders(ctx, n):
    from paper_2605_14103_amd import pf
    cfg = fdm.FeederConfig(f"feeder{n}", n_bus=n, max_depth=30, batch=6, seed=n)
    fd = _looped(cfg)
    batch = fdm.make_batch(fd, cfg)
    net = _register(ctx, fd)
    setup = ozb.zbus(fd)
    for precision, sparse in UPDATES:
        res = _solve(net, batch, precision=pf.precision(precision), zbus_sparse=sparse)
        _check(fd, batch, res, np.arange(batch.batch), f"loop{n} {precision} sparse={sparse}", setup)
    net.close()


# 255, 258, 513, 1023 and 1026 free nodes: one, two, three, four and five slots of the residual (templates of
# one, two, four and eight)
@pytest.mark.parametrize("n", [86, 87, 172, 342, 343])
def test_residual_slot_edges(ctx, n):
    from paper_2605_14103_amd import pf
    cfg = fdm.FeederConfig(f"feeder{n}", n_bus=n, max_depth=25, batch=3, seed=n)
    fd = _looped(cfg)
    batch = fdm.make_batch(fd, cfg)
    net = _register(ctx, fd)
    for precision in ("fp64", "mixed"):
        res = _solve(net, batch, precision=pf.precision(precision))
        _check(fd, batch, res, np.arange(3), f"loop{n} {precision}")
    net.close()


@pytest.mark.parametrize("precision,sparse", UPDATES)
def test_caps_zero_load_and_isolation(ctx, precision, sparse):
    import torch
    from paper_2605_14103_amd import pf
    cfg = fdm.FeederConfig("feeder40", n_bus=40, max_depth=25, batch=3, seed=41)
    fd = _looped(cfg)
    net = _register(ctx, fd)
    opts = dict(precision=pf.precision(precision), zbus_sparse=sparse)
    res = _solve(net, fdm.zero_load(fd, 3), **opts)
    assert res.converged.cpu().numpy().all() and (res.iters.cpu().numpy() == 0).all()
    # no-load voltages: rounding of Z Y_NS v_S, whose entries are below 1 pu over up to 117 terms of up to 1e3
    np.testing.assert_allclose(res.v.cpu().numpy(), np.tile(fd.v_slack, (3, fd.n_bus)), atol=1e-10)
    batch = fdm.make_batch(fd, cfg)
    capped = _solve(net, batch, zbus_max_iter=1, **opts)
    assert not capped.converged.cpu().numpy().any() and (capped.iters.cpu().numpy() == 1).all()
    bad = fdm.FeederBatch(batch.s_wye.copy(), batch.s_delta.copy())
    bad.s_wye[1, fd.wye_nodes[0]] = np.nan
    r2, full = _solve(net, bad, **opts), _solve(net, batch, **opts)
    c = r2.converged.cpu().numpy()
    assert c[0] and c[2] and not c[1]
    assert torch.equal(r2.v[0], full.v[0]) and torch.equal(r2.v[2], full.v[2])
    net.close()


@pytest.mark.parametrize("precision,sparse", UPDATES)
def test_async_enqueue_equals_host_checked(ctx, precision, sparse):
    """All iterations enqueued at once (device-side exits) against the host-checked loop, bit for
    bit: a batch, a smaller one on the same network (its counts start from zero again), and an
    iteration cap below convergence."""
    import torch
    from paper_2605_14103_amd import pf
    cfg = fdm.FeederConfig("feeder120", n_bus=120, max_depth=25, batch=300, seed=121)
    fd = _looped(cfg)
    batch = fdm.make_batch(fd, cfg)
    net = _register(ctx, fd)
    prec = pf.precision(precision)
    for b, extra in ((300, {}), (37, {}), (300, {"zbus_max_iter": 3})):
        sub = fdm.FeederBatch(batch.s_wye[:b], batch.s_delta[:b])
        ra = _solve(net, sub, precision=prec, zbus_sparse=sparse, zbus_async=1, **extra)
        rh = _solve(net, sub, precision=prec, zbus_sparse=sparse, zbus_async=0, **extra)
        for f in ("v", "iters", "converged", "mismatch", "sum_abs_change"):
            assert torch.equal(getattr(ra, f), getattr(rh, f)), f"{f} differs (batch {b}, {extra})"
        conv = ra.converged.cpu().numpy()
        assert conv.all() if not extra else not conv.any()
    _check(fd, batch, _solve(net, batch, precision=prec, zbus_sparse=sparse, zbus_async=1), spread_cols(300, 8),
           f"loop120 async {precision} sparse={sparse}")
    net.close()


@pytest.mark.parametrize("precision,sparse", UPDATES)
def test_engine_requests_equal_their_solve_alone(ctx, precision, sparse):
    from paper_2605_14103_amd import pf
    cfg = fdm.FeederConfig("feeder40", n_bus=40, max_depth=25, batch=1, seed=41)
    fd = _looped(cfg)
    net = _register(ctx, fd)
    opts = dict(precision=pf.precision(precision), zbus_sparse=sparse)
    reqs = [fdm.make_batch(fd, cfg, batch=n, seed=500 + i) for i, n in enumerate([3, 130, 1, 64, 200, 129])]
    eng = pf.Engine(net, hbm_bytes=64 << 20, n_streams=2, **opts)
    for i, b in enumerate(reqs):
        eng.submit(i, b.s_wye, b.s_delta)
    got = _collect(eng, list(range(len(reqs))))
    for i, b in enumerate(reqs):
        r = _solve(net, b, **opts)
        assert got[i].converged.all() and r.converged.cpu().numpy().all()
        assert np.array_equal(got[i].v, r.v.cpu().numpy()), f"request {i} differs from alone"
        assert np.array_equal(got[i].iters, r.iters.cpu().numpy())
    eng.close()
    net.close()


@pytest.mark.parametrize("sparse", [0, 1])
def test_caller_driven_steps(ctx, sparse):
    """One iteration per step, scenarios admitted between steps into scattered slots that are used
    again; every scenario equals its one-shot solve bit for bit."""
    import torch
    from paper_2605_14103_amd import pf
    fd = _looped(fdm.FEEDER300)
    net = _register(ctx, fd)
    batch = fdm.make_batch(fd, fdm.FEEDER300, batch=24, seed=77)
    ref = _solve(net, batch, zbus_sparse=sparse)
    v_ref, it_ref = ref.v.cpu().numpy(), ref.iters.cpu().numpy()
    eng = pf.Engine(net, hbm_bytes=1 << 30, n_streams=0, zbus_sparse=sparse)
    stream = torch.cuda.current_stream()
    free, where, got = list(range(15, -1, -2)) + list(range(0, 16, 2)), {}, {}
    waves = [range(0, 5), range(5, 9), range(9, 16), range(16, 24)]
    steps = 0
    while waves or where:
        if waves and len(free) >= len(waves[0]):
            ks = list(waves.pop(0))
            sl = [free.pop(0) for _ in ks]
            eng.admit(sl, batch.s_wye[ks], batch.s_delta[ks], stream=stream)
            where.update(zip(sl, ks))
        done, _ = eng.step(1, stream=stream)
        steps += 1
        assert steps < 200
        if done:
            r = eng.harvest(done, stream=stream)
            for j, s in enumerate(done):
                got[where.pop(s)] = (r.v[j], r.iters[j], r.converged[j])
                free.append(s)
    for k in range(24):
        v, it, ok = got[k]
        assert ok and it == it_ref[k] and np.array_equal(v, v_ref[k]), f"scenario {k} differs"
    eng.close()
    net.close()
