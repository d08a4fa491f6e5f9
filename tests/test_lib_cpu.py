"""Host-side checks of the device library that need no GPU."""
import os
import re
import subprocess

import pytest

from paper_2605_14103_amd import _lib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "pfx.h")


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(pf_[a-z0-9_]+)\s*\(", text)))


@pytest.fixture(scope="module")
def libfile():
    if not os.path.exists(_lib.LIB_PATH):
        pytest.fail("libpfx.so is not built (python -m paper_2605_14103_amd.build)")
    return _lib.LIB_PATH


def test_library_exports_every_declared_symbol(libfile):
    out = subprocess.run(["nm", "-D", "--defined-only", libfile], capture_output=True, text=True, check=True).stdout
    exported = set(line.split()[-1] for line in out.splitlines() if line.strip())
    missing = [f for f in declared_functions() if f not in exported]
    assert not missing, missing


def test_library_loads_and_binding_matches_header(libfile):
    h = _lib.lib()
    for name in declared_functions():
        assert hasattr(h, name)
    assert set(_lib.exported_names()) == set(declared_functions())


def test_defaults_and_option_struct():
    o = _lib.opts()
    assert o.precision == _lib.PF_FP64 and o.tol == 1e-8 and o.max_newton == 20
    assert o.gmres_restart == 30 and o.zbus_max_iter == 100 and o.precond_block == 0
    assert o.zbus_sparse == 0 and o.nr_direct == 0 and o.gmres_rtol == 0.0  # 0 selects the default 1e-3
    assert o.step_iters == 1 and o.zbus_async == 0 and o.forcing == 1 and o.forcing_max == 0.01
    with pytest.raises(TypeError):
        _lib.opts(not_an_option=1)


def test_ybus_builder_matches_definition():
    """The library's admittance builder on a 3-bus triangle, against the pi-model sums."""
    import ctypes

    import numpy as np

    f = np.array([0, 1, 0], dtype=np.int32)
    t = np.array([1, 2, 2], dtype=np.int32)
    r = np.array([0.01, 0.02, 0.03])
    x = np.array([0.1, 0.2, 0.3])
    b = np.array([0.02, 0.0, 0.04])
    cap = 9
    ptr = np.zeros(4, dtype=np.int32)
    col = np.zeros(cap, dtype=np.int32)
    yre = np.zeros(cap)
    yim = np.zeros(cap)
    nnz = ctypes.c_int32()
    P = lambda a: ctypes.c_void_p(a.ctypes.data)  # noqa: E731
    _lib.call("pf_tx_ybus_from_branches", 3, 3, P(f), P(t), P(r), P(x), P(b), cap, P(ptr), P(col), P(yre),
              P(yim), ctypes.byref(nnz))
    Y = np.zeros((3, 3), dtype=complex)
    for i in range(3):
        for p in range(ptr[i], ptr[i + 1]):
            Y[i, col[p]] = yre[p] + 1j * yim[p]
    ys = 1 / (r + 1j * x)
    E = np.zeros((3, 3), dtype=complex)
    for k in range(3):
        E[f[k], f[k]] += ys[k] + 0.5j * b[k]
        E[t[k], t[k]] += ys[k] + 0.5j * b[k]
        E[f[k], t[k]] -= ys[k]
        E[t[k], f[k]] -= ys[k]
    assert nnz.value == 9
    np.testing.assert_allclose(Y, E, rtol=1e-15, atol=1e-15)
    # too small a capacity is an error that still reports the needed size
    small = ctypes.c_int32()
    st = _lib.lib().pf_tx_ybus_from_branches(3, 3, P(f), P(t), P(r), P(x), P(b), 2, P(ptr), P(col), P(yre),
                                              P(yim), ctypes.byref(small))
    assert st == _lib.PF_INVALID_ARG and small.value == 9
    bad = f.copy()
    bad[0] = 7
    st = _lib.lib().pf_tx_ybus_from_branches(3, 3, P(bad), P(t), P(r), P(x), P(b), cap, P(ptr), P(col),
                                              P(yre), P(yim), ctypes.byref(small))
    assert st == _lib.PF_INVALID_ARG and b"out of range" in _lib.lib().pf_last_error()


def test_feeder_ybus_builder_matches_oracle_definition():
    """The library's three-phase builder against a dense assembly of inv(z) blocks."""
    import ctypes

    import numpy as np

    from workloads import feeder as fdm
    cfg = fdm.FeederConfig("feeder12", n_bus=12, max_depth=25, batch=1, seed=5)
    fd = fdm.make_feeder(cfg)
    n = fd.n_node
    cap = 3 * n + 18 * fd.n_seg
    ptr = np.zeros(n + 1, dtype=np.int32)
    col = np.zeros(cap, dtype=np.int32)
    yre = np.zeros(cap)
    yim = np.zeros(cap)
    nnz = ctypes.c_int32()
    z = np.ascontiguousarray(fd.z_seg)
    P = lambda a: ctypes.c_void_p(a.ctypes.data)  # noqa: E731
    _lib.call("pf_dist_ybus_from_segments", fd.n_bus, fd.n_seg, P(fd.seg_from), P(fd.seg_to), P(z), cap,
              P(ptr), P(col), P(yre), P(yim), ctypes.byref(nnz))
    Y = np.zeros((n, n), dtype=complex)
    for i in range(n):
        for p in range(ptr[i], ptr[i + 1]):
            Y[i, col[p]] = yre[p] + 1j * yim[p]
    E = np.zeros((n, n), dtype=complex)
    for s in range(fd.n_seg):
        y = np.linalg.inv(fd.z_seg[s])
        a, c = 3 * fd.seg_from[s], 3 * fd.seg_to[s]
        E[a:a + 3, a:a + 3] += y
        E[c:c + 3, c:c + 3] += y
        E[a:a + 3, c:c + 3] -= y
        E[c:c + 3, a:a + 3] -= y
    assert np.max(np.abs(Y - E)) <= 1e-12 * np.max(np.abs(E))


def _lib_ybus(grid):
    """The library's CSR of a grid's admittance matrix (host arrays)."""
    import ctypes

    import numpy as np

    P = lambda a: ctypes.c_void_p(a.ctypes.data)  # noqa: E731
    n, nb = grid.n_bus, int(grid.f.shape[0])
    cap = n + 2 * nb
    ptr = np.zeros(n + 1, dtype=np.int32)
    col = np.zeros(cap, dtype=np.int32)
    yre = np.zeros(cap)
    yim = np.zeros(cap)
    nnz = ctypes.c_int32()
    f, t = grid.f.astype(np.int32), grid.t.astype(np.int32)
    _lib.call("pf_tx_ybus_from_branches", n, nb, P(f), P(t), P(grid.r), P(grid.x), P(grid.b), cap, P(ptr),
              P(col), P(yre), P(yim), ctypes.byref(nnz))
    k = nnz.value
    return ptr, col[:k].copy(), yre[:k].copy(), yim[:k].copy()


def _switch(grid, csr, on, ldy=None):
    import ctypes

    import numpy as np

    P = lambda a: ctypes.c_void_p(a.ctypes.data)  # noqa: E731
    ptr, col, yre, yim = csr
    nnz = int(col.shape[0])
    ldy = nnz if ldy is None else ldy
    out = np.full((on.shape[0], ldy), np.nan, dtype=np.complex128)
    f, t = grid.f.astype(np.int32), grid.t.astype(np.int32)
    on = np.ascontiguousarray(on, dtype=np.uint8)
    st = _lib.lib().pf_tx_ybus_switch(grid.n_bus, nnz, P(ptr), P(col), P(yre), P(yim), int(f.shape[0]), P(f),
                                      P(t), P(grid.r), P(grid.x), P(grid.b), int(on.shape[0]), P(on), ldy,
                                      P(out))
    return st, out


def test_ybus_switch_matches_oracle_admittance():
    """Branch switching on the 30-bus grid: each scenario's values, read back as
    a dense matrix, equal the oracle's admittance matrix built from the branches
    left in service (two outages per scenario, plus the all-in-service case)."""
    import numpy as np

    from oracle import nr as onr
    from workloads import transmission as tx

    grid = tx.make_grid(tx.TX30)
    csr = _lib_ybus(grid)
    ptr, col = csr[0], csr[1]
    on = tx.make_outages(grid, 12, n_out=2, seed=5)
    on[0] = 1
    st, vals = _switch(grid, csr, on, ldy=int(col.shape[0]) + 3)
    assert st == _lib.PF_OK
    assert np.isnan(vals[:, -3:]).all()  # padding of each row untouched
    for s in range(on.shape[0]):
        Y = np.zeros((grid.n_bus, grid.n_bus), dtype=complex)
        for i in range(grid.n_bus):
            for p in range(ptr[i], ptr[i + 1]):
                Y[i, col[p]] += vals[s, p]
        m = on[s].astype(bool)
        ref = onr.ybus(grid.n_bus, grid.f[m], grid.t[m], grid.r[m], grid.x[m], grid.b[m]).toarray()
        np.testing.assert_allclose(Y, ref, rtol=0, atol=1e-12 * np.abs(ref).max())
    # all in service: the base values exactly
    np.testing.assert_array_equal(vals[0, :col.shape[0]], csr[2] + 1j * csr[3])


def test_ybus_switch_errors():
    import ctypes

    import numpy as np

    from workloads import transmission as tx

    grid = tx.make_grid(tx.TX30)
    csr = _lib_ybus(grid)
    on = np.ones((2, grid.f.shape[0]), dtype=np.uint8)
    st, _ = _switch(grid, csr, on, ldy=int(csr[1].shape[0]) - 1)
    assert st == _lib.PF_INVALID_ARG and b"ldy" in _lib.lib().pf_last_error()
    # a branch whose entries are not in the pattern
    import dataclasses
    f = grid.f.copy()
    t = grid.t.copy()
    pairs = set(zip(f.tolist(), t.tolist())) | set(zip(t.tolist(), f.tolist()))
    a, c = next((i, j) for i in range(grid.n_bus) for j in range(grid.n_bus) if i != j and (i, j) not in pairs)
    f[0], t[0] = a, c
    g2 = dataclasses.replace(grid, f=f, t=t)
    st, _ = _switch(g2, csr, on)
    assert st == _lib.PF_INVALID_ARG and b"pattern" in _lib.lib().pf_last_error()
    # zero scenarios is a no-op
    st, out = _switch(grid, csr, on[:0])
    assert st == _lib.PF_OK and out.shape[0] == 0
    del ctypes


def _compile_and_run(tmp_path, code):
    """Build a small program over the library's host headers with g++ and return its output lines."""
    src, exe = tmp_path / "probe.cpp", tmp_path / "probe"
    src.write_text(code)
    subprocess.run(["g++", "-std=c++17", "-O2", f"-I{os.path.join(ROOT, 'paper_2605_14103_amd', 'csrc')}", str(src),
                    "-o", str(exe)], check=True, capture_output=True, text=True)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split("\n")[:-1]


def test_direct_step_allocation_agrees_with_launch(tmp_path):
    """The direct step's caller allocates device memory for the factor values by the unsplit
    workgroup's LDS; the launch must then take a split that keeps them where the caller expects
    them.  Every count of doubles across the 160 KB boundary, for each workgroup shape and wish."""
    shapes = [(64, 1, 1), (256, 1, 4), (1024, 4, 4), (2048, 4, 4)]   # bus positions, waves, largest split
    code = "#include <cstdio>\n#include \"direct.hpp\"\nusing namespace pfx;\nint main() {\n"
    for nbp, waves, most in shapes:
        code += (f"  for (int v = 20480 - {4 * nbp} - 80; v < 20480 - {4 * nbp} + 8; ++v)\n"
                 "    for (int want : {0, 1, 2, 3, 4, 16}) {\n"
                 f"      const int s = direct_fitting_split({nbp}, {waves}, v - 100, 50, want, {most});\n"
                 f"      printf(\"{nbp} {waves} {most} %d %d %d %d %zu\\n\", v, want, s,\n"
                 f"             (int)direct_in_lds({nbp}, {waves}, v - 100, 50),\n"
                 f"             direct_lds_bytes({nbp}, s * {waves}, v - 100, 50));\n    }}\n")
    lines = _compile_and_run(tmp_path, code + "}\n")
    narrowed = 0
    for line in lines:
        nbp, waves, most, v, want, s, in_lds, launched = (int(x) for x in line.split())
        assert in_lds == (32 * nbp + 16 * waves + 8 * v <= 163840)   # as the caller decides
        assert launched == 32 * nbp + 16 * waves * s + 8 * v and (launched <= 163840) == bool(in_lds)
        wish = max(k for k in (1, 2, 4) if k <= max(1, min(want, most)))
        assert s == wish or (s < wish and in_lds and launched + 16 * waves * s > 163840)
        narrowed += s < wish
    assert len(lines) == 4 * 88 * 6 and narrowed > 0


def test_solver_lds_grew_for_no_unsplit_grid(tmp_path):
    """LDS of the Newton and adjoint kernels over every core size and restart: the core's right-hand
    side with its zeros lies within the layout and clear of everything live beside it, and an unsplit
    workgroup of the largest grids takes no more than the right-hand side in whole fours needs, so
    that none is refused for the zeros."""
    shapes = [(64, 1, 1), (256, 1, 4), (1024, 4, 4), (2048, 4, 4), (4096, 8, 2), (8192, 16, 1)]
    code = "#include <cstdio>\n#include \"nr_layout.hpp\"\nusing namespace pfx;\nint main() {\n"
    for nbp, waves, most in shapes:
        code += (f"  for (int s = 1; s <= {most}; s *= 2) for (int ts = 4; ts <= 8; ts += 4)\n"
                 "    for (int k = 0; k <= 2048; ++k) for (int R = 1; R <= 64; ++R) {\n"
                 f"      const NrLayout L = nr_layout({nbp}, {nbp - 1}, {nbp - 1}, k, R, s * {waves}, s > 1, ts);\n"
                 "      const int end = L.tmp + core_entries(k, ts) * ts;\n"
                 "      // whole part within its own area (the partials', or its own), zeros before H\n"
                 "      const bool inside = L.tmp + (k + 3) / 4 * 4 * ts <= L.redn && end <= L.H;\n"
                 f"      int old = 16 * {nbp}, red = 16 * (R + 2) * {waves}, core = ((k ? k : 1) + 3) / 4 * 4 * ts;\n"
                 f"      old += red + (core > red ? align16(core) : 0) + align16(8 * {waves}) + align16(R * (R + 1) / 2 * ts);\n"
                 "      old += 4 * align16(R * ts) + align16((R + 1) * ts);\n"
                 f"      if (!inside || (old <= 163840 && L.total > 163840) || ({waves} >= 8 && s == 1 && L.total > old))\n"
                 f"        printf(\"{nbp} %d %d %d %d: %d, before %d, inside %d\\n\", s, ts, k, R, L.total, old, (int)inside);\n"
                 "    }\n")
    assert _compile_and_run(tmp_path, code + "}\n") == []
