"""Which feeders take the tree form of the solve.  A feeder that differs from a
radial one without shunts in any one respect keeps the general forms, and is
solved for what it is: each against a dense fixed point in numpy from the same
admittance matrix."""
import ctypes

import numpy as np
import pytest

from oracle import zbus as ozb
from tests.gpu_common import to_dev

pytestmark = pytest.mark.gpu

A = np.exp(-2j * np.pi / 3)
V_SLACK = np.array([1.0, A, A * A])


class Case:
    """A feeder by its admittance matrix; changed by the tests before it is solved."""

    def __init__(self, n, seed=0):
        rng = np.random.default_rng(seed)
        self.n = n
        self.segments = [(int(rng.integers(0, k)), k) for k in range(1, n)]
        self.z = []
        for _ in self.segments:
            k = rng.uniform(0.3, 0.5, 3)
            z = np.eye(3, dtype=complex)
            for (a, b), c in zip(((0, 1), (1, 2), (2, 0)), k):
                z[a, b] = z[b, a] = c
            self.z.append(z * (rng.uniform(0.1, 0.6) + 1j * rng.uniform(0.2, 0.8)) * 0.01)
        self.Y = np.zeros((3 * n, 3 * n), dtype=complex)
        for (a, c), z in zip(self.segments, self.z):
            self.add_segment(a, c, z)
        self.slack = [0, 1, 2]
        kind = rng.integers(0, 4, n)
        kind[0] = 0
        kind[1:4] = (1, 2, 3)[:n - 1]
        s = rng.uniform(0.2, 1.0, 3 * n) * (1 + 0.3j) / n
        per = np.repeat(kind, 3)
        self.s_wye, self.s_delta = np.where(per & 1, s, 0), np.where(per & 2, s[::-1], 0)
        self.delta = [[3 * b, 3 * b + 1, 3 * b + 2] for b in range(n) if kind[b] & 2]

    def add_segment(self, a, c, z):
        y = np.linalg.inv(z)
        y = (y + y.T) / 2
        i, j = np.arange(3 * a, 3 * a + 3), np.arange(3 * c, 3 * c + 3)
        for p, q, w in ((i, i, y), (j, j, y), (i, j, -y), (j, i, -y)):
            self.Y[np.ix_(p, q)] += w

    def relabel(self, to):
        """Node k becomes node to[k]."""
        back = np.argsort(to)
        self.Y = self.Y[np.ix_(back, back)]
        self.s_wye, self.s_delta = self.s_wye[back], self.s_delta[back]
        self.slack = [int(to[k]) for k in self.slack]
        self.delta = [[int(to[k]) for k in d] for d in self.delta]

    def solve(self, **opts):
        """(voltages, converged, bytes held by the registered feeder)"""
        import torch
        from paper_2605_14103_amd import _lib as L
        from paper_2605_14103_amd import pf
        N = self.Y.shape[0]
        rows, cols = np.nonzero(self.Y)
        ptr = np.zeros(N + 1, dtype=np.int32)
        ptr[1:] = np.cumsum(np.bincount(rows, minlength=N))
        col = cols.astype(np.int32)
        vals = self.Y[rows, cols]
        yre, yim = np.ascontiguousarray(vals.real), np.ascontiguousarray(vals.imag)
        sl, vs = np.array(self.slack, dtype=np.int32), V_SLACK.copy()
        wy = np.flatnonzero(self.s_wye).astype(np.int32)
        de = np.array(self.delta, dtype=np.int32).reshape(-1, 3)
        P = lambda a: ctypes.c_void_p(a.ctypes.data)  # noqa: E731
        ctx = pf.Context(0)
        net = pf.DistNetwork.__new__(pf.DistNetwork)
        net.ctx, net.n_node, net.h = ctx, N, ctypes.c_void_p()
        o = L.opts()
        try:
            L.call("pf_dist_network_create", ctx.h, N, len(col), P(ptr), P(col), P(yre), P(yim), P(sl), P(vs),
                   len(wy), P(wy), len(de), P(de), ctypes.byref(o), ctypes.byref(net.h))
            held = ctx.bytes()
            res = net.solve(to_dev(self.s_wye[None, :]), to_dev(self.s_delta[None, :]), **opts)
            torch.cuda.synchronize()
            return res.v.cpu().numpy()[0], bool(res.converged[0]), held
        finally:
            net.close()
            ctx.close()

    def reference(self):
        N = np.setdiff1d(np.arange(self.Y.shape[0]), self.slack)
        pos = -np.ones(self.Y.shape[0], dtype=int)
        pos[N] = np.arange(len(N))
        Z = np.linalg.inv(self.Y[np.ix_(N, N)])
        v0 = -Z @ (self.Y[np.ix_(N, self.slack)] @ V_SLACK)
        d = pos[np.array(self.delta, dtype=int).reshape(-1, 3)]
        v = v0[:, None]
        sw, sd = self.s_wye[N][:, None], self.s_delta[N][:, None]
        for _ in range(60):
            v = Z @ ozb.injection(v, sw, sd, d) + v0[:, None]
        out = np.zeros(self.Y.shape[0], dtype=complex)
        out[self.slack] = V_SLACK
        out[N] = v[:, 0]
        return out


def _is_general(held, n_free):
    # Z in two precisions, at least 2 n_free rows of a multiple of 128 columns; the tree's tables are below 450
    # bytes for each of its buses (64 at least)
    return held >= 12 * (2 * n_free) * 128


def _shunt(f):
    f.Y[np.arange(15, 18), np.arange(15, 18)] += 0.02j


def _charging(f):
    for b in f.segments[4]:
        f.Y[np.arange(3 * b, 3 * b + 3), np.arange(3 * b, 3 * b + 3)] += 1e-6j


def _ground(f):   # a shunt between two phases: no change of the row's own magnitude sum in sight
    f.Y[15, 16] += 0.01
    f.Y[16, 15] += 0.01


def _unsymmetric(f):
    a, c = f.segments[5]
    for i, j, s in ((a, a, 1), (c, c, 1), (a, c, -1), (c, a, -1)):
        f.Y[3 * i, 3 * j + 1] += s * 0.4


def _not_mirrored(f):
    a, c = f.segments[5]
    f.Y[3 * a, 3 * c] += 0.4
    f.Y[3 * a, 3 * a] -= 0.4


def _phase_shift(f):
    a, c = f.segments[5]
    e = np.exp(0.02j)
    f.Y[3 * a:3 * a + 3, 3 * c:3 * c + 3] *= e
    f.Y[3 * c:3 * c + 3, 3 * a:3 * a + 3] *= e.conjugate()


def _loop(f):
    f.add_segment(2, 11, f.z[0])


def _delta_over_two_buses(f):
    b, c = f.delta[0], f.delta[1]
    b[2], c[2] = c[2], b[2]


def _delta_order(f):
    f.delta[0] = [f.delta[0][i] for i in (0, 2, 1)]


def _delta_turned(f):   # the same load, named from another phase on: b, c, a
    f.delta[0] = [f.delta[0][i] for i in (1, 2, 0)]


def _phases_swapped(f):
    to = np.arange(3 * f.n)
    to[[15, 16]] = to[[16, 15]]
    f.relabel(to)


def _nodes_shuffled(f):
    f.relabel(np.random.default_rng(1).permutation(3 * f.n))


def _slack_order(f):
    f.slack = [0, 2, 1]


def _two_phase_lateral(f):   # a leaf of two phases: the last bus without its third node
    b = f.n - 1
    a = f.segments[b - 1][0]
    f.Y[3 * b:, :] = 0
    f.Y[:, 3 * b:] = 0
    f.Y[3 * a:3 * a + 3, 3 * a:3 * a + 3] = -sum(f.Y[3 * a:3 * a + 3, 3 * c:3 * c + 3] for c in range(b) if c != a)
    y = np.linalg.inv(f.z[-1][:2, :2])
    i, j = np.arange(3 * a, 3 * a + 2), np.arange(3 * b, 3 * b + 2)
    for p, q, w in ((i, i, y), (j, j, y), (i, j, -y), (j, i, -y)):
        f.Y[np.ix_(p, q)] += w
    f.Y = f.Y[:-1, :-1]
    f.s_wye, f.s_delta = f.s_wye[:-1], f.s_delta[:-1]
    f.delta = [d for d in f.delta if d[0] != 3 * b]


def _parallel(f):
    f.add_segment(*f.segments[5], f.z[0])


# tol 1e-11 over at most 36 nodes and impedances below 0.2 moves no voltage by 1e-9
@pytest.mark.parametrize("change,general", [
    (None, False), (_parallel, False), (_shunt, True), (_charging, True), (_ground, True), (_loop, True),
    (_delta_over_two_buses, True), (_delta_order, True), (_delta_turned, False), (_phases_swapped, True),
    (_nodes_shuffled, True), (_slack_order, True), (_two_phase_lateral, True)], ids=lambda c: c.__name__[1:] if callable(c) else str(c))
@pytest.mark.parametrize("sparse", [0, 1])
def test_one_difference_keeps_the_general_form(change, general, sparse):
    f = Case(12)
    if change:
        change(f)
    v, ok, held = f.solve(tol=1e-11, zbus_sparse=sparse)
    assert ok
    np.testing.assert_allclose(v, f.reference(), rtol=0, atol=1e-9)
    assert _is_general(held, f.Y.shape[0] - 3) == general


@pytest.mark.parametrize("change", [_unsymmetric, _not_mirrored, _phase_shift])
def test_unsymmetric_feeders_stay_refused(change):
    """No form solves a feeder whose admittance matrix is not symmetric."""
    from paper_2605_14103_amd import _lib as L
    f = Case(12)
    change(f)
    with pytest.raises(L.PfError) as e:
        f.solve()
    assert e.value.status == L.PF_SINGULAR_SETUP


@pytest.mark.parametrize("z", [1e-12, 1e-14])
def test_too_stiff_feeders_stay_refused(z):
    """Segments so short beside the others that the admittance matrix's rounding alone exceeds the
    solver's tolerance are reported when the feeder is registered, as for the general form, and not
    by solves that never converge."""
    from paper_2605_14103_amd import _lib as L
    f = Case(30)
    f.Y[:] = 0
    for k, (a, c) in enumerate(f.segments):
        f.add_segment(a, c, z / 0.01 * f.z[k] if k % 5 == 4 else f.z[k])
    with pytest.raises(L.PfError) as e:
        f.solve()
    assert e.value.status == L.PF_SINGULAR_SETUP


@pytest.mark.parametrize("b_shunt", [2e-7, 0.0])
def test_small_shunt_behind_a_closed_switch(b_shunt):
    """A closed switch (1e-7 pu) with 2e-7 pu of charging behind it, no load: the shunt lies far
    below the rounding of the switch's admittance in magnitude, but is there exactly in the
    admittance matrix (in the part of it that the switch leaves alone), and moves the voltage by
    1e-7.  Without it the same feeder is a tree."""
    f = Case(3)
    z1 = 0.2 + 0.4j
    f.Y[:] = 0
    f.add_segment(0, 1, z1 * np.eye(3))
    f.add_segment(1, 2, 1e-7 * np.eye(3))
    f.Y[range(6, 9), range(6, 9)] += 1j * b_shunt
    f.s_wye[:], f.s_delta[:] = 0, 0
    f.delta = []
    v, ok, held = f.solve()
    assert ok
    y = 1j * b_shunt
    want = V_SLACK / (1 + y * (z1 + 1e-7))
    # condition of the admittance matrix (2e7 pu over 0.45 pu) times the unit roundoff, and a factor of 20
    np.testing.assert_allclose(v[6:], want, rtol=0, atol=2e-8)
    assert _is_general(held, 6) == (b_shunt != 0)
