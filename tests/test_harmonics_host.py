"""The generated solid-harmonic expansion code (the GPU kernels' arithmetic,
built here for the host with T = double) against the oracle's Cartesian
formulas."""
import ctypes
import math
import os
import subprocess
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1310_4502_amd", "csrc")
SIZE = 400  # more than any coefficient row


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("harm"))
    gen = os.path.join(out, "harmonics.h")
    subprocess.run([sys.executable, os.path.join(CSRC, "gen_harmonics.py"), gen], check=True)
    lib = os.path.join(out, "libharm.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-ffp-contract=off", "-fPIC", "-shared", "-I", out,
                    os.path.join(ROOT, "tests", "host", "harmonics_shim.cpp"), "-o", lib],
                   check=True)
    L = ctypes.CDLL(lib)
    i, v, d = ctypes.c_int, ctypes.c_void_p, ctypes.c_double
    L.shim_fwd.argtypes = [i, i, v, v, v, d, v]
    L.shim_sink.argtypes = [i, i, v, v, v, d, v, v]
    L.shim_cell.argtypes = [i, v, d, v, v]
    L.shim_coef.argtypes = [i, i, v, v, v]
    L.shim_coefT.argtypes = [i, v, v]
    return L


def P(a):
    return a.ctypes.data_as(ctypes.c_void_p)


def coef(shim, p, M, hess=0):
    h, t = np.full(SIZE, np.nan), np.full(SIZE, np.nan)
    shim.shim_coef(p, hess, P(M), P(h), P(t))
    return h, t


MODES = [("plummer", 0.0, 0), ("plummer", 0.0, 1), ("plummer", 0.4, 1), ("k1", 2.5, 2)]


@pytest.mark.parametrize("p", range(9))
@pytest.mark.parametrize("kernel,eps,mode", MODES)
def test_forward_matches_oracle(orc, shim, p, kernel, eps, mode):
    """Field and potential; K1 with half of the points inside its radius."""
    rng = np.random.default_rng(p)
    M = orc.p2m(p, rng.random((30, 3)) - 0.5, rng.random(30), np.zeros(3))
    h, t = coef(shim, p, M)
    for k in range(8):
        R = rng.normal(size=3) * (3 if k % 2 == 0 else 0.8)
        out = np.zeros(4)
        shim.shim_fwd(p, mode, P(h), P(t), P(R), eps * eps, P(out))
        a, phi = orc.m2p(p, M, R, eps, kernel=kernel)
        # the oracle's terms grow towards the cell: round-off of its own sum
        tol = 1e-12 * (1 + 1e3 * (np.linalg.norm(R) < 1))
        assert np.abs(-out[:3] - a).max() <= tol * np.abs(a).max()
        assert abs(out[3] - phi) <= tol * max(abs(phi), 1e-2)


@pytest.mark.parametrize("p", range(9))
@pytest.mark.parametrize("kernel,eps,mode", MODES)
def test_sink_adjoint_is_the_fields_jacobian(orc, shim, p, kernel, eps, mode):
    """g_l = sum_k b_k d(field_k)/dx_l by fourth-order differences of the
    oracle's expansion: step 1e-3 leaves 1e-12 of truncation and 1e-12 of
    rounding per term, 1e-8 covers both where terms grow towards the cell."""
    rng = np.random.default_rng(50 + p)
    M = orc.p2m(p, rng.random((30, 3)) - 0.5, rng.random(30), np.zeros(3))
    h, t = coef(shim, p, M, 1)
    for k in range(6):
        d = rng.normal(size=3)
        # clear of the kernel edge, where the order-4 radial derivative jumps
        R = d / np.linalg.norm(d) * (3.5 if k % 2 == 0 else 1.7)
        b = rng.normal(size=3)
        g = np.zeros(3)
        shim.shim_sink(p, mode, P(h), P(t), P(R), eps * eps, P(b), P(g))

        def psi(x):
            return -float(np.dot(b, orc.m2p(p, M, x, eps, kernel=kernel)[0]))

        s = 2e-3
        ref = np.zeros(3)
        for i in range(3):
            e = np.zeros(3)
            e[i] = s
            ref[i] = (8 * (psi(R + e) - psi(R - e)) - (psi(R + 2 * e) - psi(R - 2 * e))) / (12 * s)
        assert np.abs(g - ref).max() <= 1e-8 * np.abs(ref).max()


@pytest.mark.parametrize("p", range(9))
def test_cell_rows_and_their_transpose(orc, shim, p):
    """<b, field(C)> = <row(b), C> for Newtonian multipoles, and the transposed
    coefficient map is the adjoint of the map itself."""
    rng = np.random.default_rng(80 + p)
    nm = (p + 1) * (p + 2) * (p + 3) // 6
    M = rng.normal(size=nm)
    h, t = coef(shim, p, M)
    n = 1 + 3 * p * p
    assert np.isfinite(h[:n]).all() and np.isnan(h[n:]).all()
    for _ in range(4):
        R = rng.normal(size=3) * 2
        b = rng.normal(size=3)
        out, row = np.zeros(4), np.zeros(SIZE)
        shim.shim_fwd(p, 0, P(h), P(t), P(R), 0.09, P(out))
        shim.shim_cell(p, P(R), 0.09, P(b), P(row))
        terms = row[:n] * h[:n]
        assert abs(np.dot(b, out[:3]) - terms.sum()) <= 1e-13 * np.abs(terms).sum() + 1e-300
        back = np.zeros(nm)
        shim.shim_coefT(p, P(row), P(back))
        assert abs(np.dot(back, M) - terms.sum()) <= 1e-12 * np.abs(back * M).sum()


@pytest.mark.parametrize("p", range(2, 9))
def test_newtonian_rule_bounds_what_it_leaves_out(orc, shim, p):
    """Where the kernels take the Newtonian multipoles under Plummer softening
    they leave out at most kNewtonC eps^2 b^2 / (d - b)^4 of the cell's
    monopole field: checked on point masses at distance b (the worst case, of
    which every cell is a positive sum) over separations and directions."""
    import re
    src = open(os.path.join(CSRC, "common.h")).read()
    c = float(re.search(r"kNewtonC = ([0-9.]+)", src).group(1))
    rng = np.random.default_rng(7)
    eps, b, worst = 1e-3, 0.5, 0.0
    for ratio in (1.05, 1.3, 1.7, 2.0, 2.5, 4.0, 8.0):
        for _ in range(40):
            d = rng.normal(size=3)
            pt = d / np.linalg.norm(d) * b
            e = rng.normal(size=3)
            if _ < 8:
                e = d * (1 if _ % 2 else -1) + 0.1 * e  # along and against the offset
            R = e / np.linalg.norm(e) * b * ratio
            M = orc.p2m(p, pt[None, :], np.ones(1), np.zeros(3))
            h, t = coef(shim, p, M)
            full, newt = np.zeros(4), np.zeros(4)
            shim.shim_fwd(p, 1, P(h), P(t), P(R), eps * eps, P(full))
            shim.shim_fwd(p, 0, P(h), P(t), P(R), eps * eps, P(newt))
            r = np.linalg.norm(R)
            rel = np.linalg.norm(full[:3] - newt[:3]) * r * r
            worst = max(worst, rel / (eps * eps * b * b / (r - b) ** 4))
    assert worst <= c, worst


def newton_constant(name):
    import re
    return float(re.search(name + r" = ([0-9.]+)", open(os.path.join(CSRC, "common.h")).read()).group(1))


@pytest.mark.parametrize("p", range(2, 9))
@pytest.mark.parametrize("ratio", [1.05, 1.3, 1.7, 2.0, 2.5, 4.0, 10.0, 60.0])
def test_newtonian_rules_of_the_derivatives(orc, shim, p, ratio):
    """What Newtonian multipoles leave out of a unit mass's field, as derivatives
    by the sink's position (kNewtonCH eps^2 b^2 / (d - b)^4 of the monopole's
    2 / d^3) and by the mass's own (kNewtonCS eps^2 b d / (d - b)^4, for every
    softening; its mass gradient, the field itself, is within that too)."""
    ch, cs = newton_constant("kNewtonCH"), newton_constant("kNewtonCS")
    rng = np.random.default_rng(11)
    idx = np.array(orc.multi_indices(p))
    b, worst_h, worst_s, worst_m = 0.5, 0.0, 0.0, 0.0

    def left_out(M, R, e2):
        h, t = coef(shim, p, np.ascontiguousarray(M))
        full, newt = np.zeros(4), np.zeros(4)
        shim.shim_fwd(p, 1, P(h), P(t), P(R), e2, P(full))
        shim.shim_fwd(p, 0, P(h), P(t), P(R), e2, P(newt))
        return full[:3] - newt[:3]

    for trial in range(24):
        u, e = rng.normal(size=3), rng.normal(size=3)
        if trial < 10:
            e = u * (1 if trial % 2 else -1) + 0.1 * e  # along and against the offset
        x, d = u / np.linalg.norm(u) * b, b * ratio
        R = e / np.linalg.norm(e) * d
        M = np.prod(x ** idx, axis=1)
        for eps in (1e-3 * b, 0.1 * b, b):
            e2 = eps * eps
            unit = e2 / (d - b) ** 4
            h, t = coef(shim, p, M, 1)
            J = np.zeros((3, 3))
            for k in range(3):
                bar, full, newt = np.eye(3)[k], np.zeros(3), np.zeros(3)
                shim.shim_sink(p, 1, P(h), P(t), P(R), e2, P(bar), P(full))
                shim.shim_sink(p, 0, P(h), P(t), P(R), e2, P(bar), P(newt))
                J[k] = full - newt
            worst_h = max(worst_h, np.linalg.norm(J, 2) * d ** 3 / 2 / (unit * b * b))
            S = np.zeros((3, 3))
            for k in range(3):
                low = idx.copy()
                low[:, k] = np.maximum(low[:, k] - 1, 0)
                S[k] = left_out(idx[:, k] * np.prod(x ** low, axis=1), R, e2)
            worst_s = max(worst_s, np.linalg.norm(S, 2) * d ** 3 / 2 / (unit * b * d))
            worst_m = max(worst_m, np.linalg.norm(left_out(M, R, e2)) * d * d / (unit * b * d))
    assert worst_h <= ch and worst_s <= cs and worst_m <= cs, (worst_h, worst_s, worst_m)


def test_benchmark_counts_the_generated_operations():
    """The operation counts of the benchmark's rates are those of the emitted
    expressions (order 0 without the terms that vanish there)."""
    sys.path.insert(0, CSRC)
    sys.path.insert(0, ROOT)
    import bench
    import gen_harmonics as g
    for p in range(9):
        if p > 0:
            assert bench.flops_m2p(p) == g.flops("field", p)
        assert bench.flops_m2p_sink_adj(p) == g.flops("jacobian", p)
        assert bench.flops_m2p_cell_adj(p) == g.flops("cell", p)
