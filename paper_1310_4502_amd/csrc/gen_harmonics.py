#!/usr/bin/env python3
"""Generate straight-line HIP code for the cell-body expansion in solid
harmonics.

The order-n part of the expansion is M_n(d) G with the homogeneous symbol
M_n(xi) = sum_{|alpha|=n} w_alpha M_alpha xi^alpha. Split into harmonic parts,
    M_n(xi) = sum_k |xi|^(2k) h_{l,k}(xi),   l = n - 2k,  h_{l,k} harmonic,
and a harmonic operator acts on a radial function by Hobson's theorem,
    h_l(d) f(|R|^2) = h_l(R) (2 d/ds)^l f,
so the sum of C(p+4,3) Cartesian derivatives becomes, per degree, one harmonic
polynomial times one radial function. With F_n = (2 d/ds)^n f:
    sum_alpha w M d^alpha G = sum_{l,k} h_{l,k}(R) g_{l,k},
    g_{l,k} = (Laplacian in 3 + 2l dimensions)^k F_l,   (2 d/ds) g_{l,k} = g_{l+1,k}.
The trace parts (k >= 1) vanish for the Newtonian kernel.

Coefficients of one cell, in the order the kernels read them (harmonic part;
degree-l block at 1 + 3 (l-1)^2):
    [H_0] and for l = 1 .. p the 3 (2l-1) coefficients of grad H_l in the basis
    Y_{l-1,m} (m = 0, 1c, 1s, 2c, ..), x y z together per m,
with H_l = (-1)^(l+1) (2l-1)!! h_l, so that the Plummer radial functions become
the plain powers u^(2n+1), u = (|R|^2 + e^2)^(-1/2). H_l itself is
R . grad H_l / l. The trace part holds the same for k >= 1, by n = l + 2k, then
k (a single coefficient for l = 0). A prefix of either serves a lower order.
The sink-side adjoint reads second derivatives instead: [H_0], grad H_1, and for
l = 2 .. p the 5 (2l-3) coefficients of (xx, xy, xz, yy, yz) of the Hessian of
H_l in the basis Y_{l-2,m} (zz = -xx - yy), block at 4 + 5 (l-2)^2.

The basis is Y_{l,m} = P_{l,m}(z, rho) {Re, Im} (x + i y)^m with P monic in z,
    Y_{l,l} = {Re, Im} (x + i y)^l,  Y_{l,m} = z Y_{l-1,m} - c_lm rho Y_{l-2,m},
    c_lm = ((l-1)^2 - m^2) / ((2l-1)(2l-3)),  rho = |R|^2.
"""
import os
import sys
from fractions import Fraction as Fr
from functools import lru_cache
from math import comb, factorial

PMAX = 8


def lit(x):
    return f"T({float(x)!r})"


def dfact(n):
    r = 1
    while n > 1:
        r *= n
        n -= 2
    return r


# ------------------------------------------------------------ polynomials
def padd(p, q, s=Fr(1)):
    r = dict(p)
    for k, v in q.items():
        r[k] = r.get(k, Fr(0)) + s * v
        if r[k] == 0:
            del r[k]
    return r


def pmul(p, q):
    r = {}
    for (a, b, c), v in p.items():
        for (d, e, f), w in q.items():
            k = (a + d, b + e, c + f)
            r[k] = r.get(k, Fr(0)) + v * w
    return {k: v for k, v in r.items() if v}


def pdiff(p, i):
    r = {}
    for k, v in p.items():
        if k[i]:
            e = list(k)
            e[i] -= 1
            r[tuple(e)] = r.get(tuple(e), Fr(0)) + v * k[i]
    return r


X, Y, Z = {(1, 0, 0): Fr(1)}, {(0, 1, 0): Fr(1)}, {(0, 0, 1): Fr(1)}
RHO = {(2, 0, 0): Fr(1), (0, 2, 0): Fr(1), (0, 0, 2): Fr(1)}


def clm(l, m):
    return Fr((l - 1) ** 2 - m * m, (2 * l - 1) * (2 * l - 3))


@lru_cache(None)
def _basis(l, m, s):
    if m == l:
        if l == 0:
            return {(0, 0, 0): Fr(1)}
        if l == 1:
            return Y if s else X
        c, d = _basis(l - 1, l - 1, 0), _basis(l - 1, l - 1, 1)
        return padd(pmul(X, d), pmul(Y, c)) if s else padd(pmul(X, c), pmul(Y, d), Fr(-1))
    p = pmul(Z, _basis(l - 1, m, s))
    if m <= l - 2:
        p = padd(p, pmul(RHO, _basis(l - 2, m, s)), -clm(l, m))
    return p


def harmonics(l):
    """(m, s) of the degree-l basis: s = 0 the real, 1 the imaginary part."""
    return [(0, 0)] + [(m, s) for m in range(1, l + 1) for s in (0, 1)]


def monomials(n):
    """Exponents of order n in moment slot order."""
    return [(a, b, n - a - b) for a in range(n, -1, -1) for b in range(n - a, -1, -1)]


@lru_cache(None)
def decompose(n):
    """{(k, m, s): {alpha: coefficient}}: the coefficient of |xi|^(2k) Y_{n-2k,m,s}
    in the monomial xi^alpha."""
    mono = monomials(n)
    cols, tags = [], []
    for k in range(n // 2 + 1):
        r2k = {(0, 0, 0): Fr(1)}
        for _ in range(k):
            r2k = pmul(r2k, RHO)
        for m, s in harmonics(n - 2 * k):
            cols.append(pmul(r2k, _basis(n - 2 * k, m, s)))
            tags.append((k, m, s))
    N = len(mono)
    A = [[cols[j].get(mono[i], Fr(0)) for j in range(N)] +
         [Fr(1) if i == j else Fr(0) for j in range(N)] for i in range(N)]
    for i in range(N):
        piv = next(r for r in range(i, N) if A[r][i])
        A[i], A[piv] = A[piv], A[i]
        d = A[i][i]
        A[i] = [v / d for v in A[i]]
        for r in range(N):
            if r != i and A[r][i]:
                f = A[r][i]
                A[r] = [v - f * w if w else v for v, w in zip(A[r], A[i])]
    return {tags[j]: {mono[i]: A[j][N + i] for i in range(N) if A[j][N + i]} for j in range(N)}


def in_basis(poly, l):
    """Coefficients of a harmonic polynomial of degree l in the basis."""
    d = decompose(l)
    out = {}
    for k, m, s in d:
        v = sum((poly.get(al, Fr(0)) * c for al, c in d[(k, m, s)].items()), Fr(0))
        assert k == 0 or v == 0
        if k == 0:
            out[(m, s)] = v
    return out


@lru_cache(None)
def gradient(l, m, s, i):
    return in_basis(pdiff(_basis(l, m, s), i), l - 1)


HESS = [(0, 0), (0, 1), (0, 2), (1, 1), (1, 2)]


@lru_cache(None)
def hessian(l, m, s, q):
    i, j = HESS[q]
    return in_basis(pdiff(pdiff(_basis(l, m, s), i), j), l - 2)


def weight(al):
    return Fr((-1) ** sum(al), factorial(al[0]) * factorial(al[1]) * factorial(al[2]))


def norm(l):
    """H_l = norm(l) h_l."""
    return Fr((-1) ** (l + 1) * dfact(2 * l - 1))


# ------------------------------------------------------------ coefficient layout
def off_h(l):
    return 0 if l == 0 else 1 + 3 * (l - 1) ** 2


def off_t(l, k):
    """Offset of the (l, k) block, k >= 1, in the trace part."""
    o = 0
    for n in range(2, PMAX + 1):
        for kk in range(1, n // 2 + 1):
            if (n - 2 * kk, kk) == (l, k):
                return o
            o += size_grad(n - 2 * kk)
    raise KeyError((l, k))


def size_grad(l):
    return 1 if l == 0 else 3 * (2 * l - 1)


def off_hh(l):
    return {0: 0, 1: 1}.get(l, 4 + 5 * (l - 2) ** 2)


def size_hess(l):
    return {0: 1, 1: 3}.get(l, 5 * (2 * l - 3))


def off_th(l, k):
    o = 0
    for n in range(2, PMAX + 1):
        for kk in range(1, n // 2 + 1):
            if (n - 2 * kk, kk) == (l, k):
                return o
            o += size_hess(n - 2 * kk)
    raise KeyError((l, k))


def block_map(l, k, hess):
    """[{alpha: literal}] per coefficient of the (l, k) block, from the raw
    moments of order l + 2k (expansion weight folded in)."""
    n = l + 2 * k
    d = decompose(n)
    if l == 0:
        return [{al: norm(0) * c * weight(al) for al, c in d[(k, 0, 0)].items()}]
    rows = []
    if hess and l >= 2:
        deg, comps, fn = l - 2, 5, hessian
    else:
        deg, comps, fn = l - 1, 3, gradient
    for mo, so in harmonics(deg):
        for i in range(comps):
            r = {}
            for m, s in harmonics(l):
                g = fn(l, m, s, i)[(mo, so)]
                if g:
                    for al, c in d[(k, m, s)].items():
                        r[al] = r.get(al, Fr(0)) + norm(l) * g * c * weight(al)
            rows.append({al: v for al, v in r.items() if v})
    return rows


def gen_coef(n, hess):
    """Coefficients of every (l, k) block with l + 2k = n from the order-n raw
    moments M (slot order within the order), scaled by sc = side^-n."""
    slots = {al: i for i, al in enumerate(monomials(n))}
    L = []
    for k in range(n // 2 + 1):
        l = n - 2 * k
        if hess:
            base = f"h[{off_hh(l)} + " if k == 0 else f"t[{off_th(l, k)} + "
        else:
            base = f"h[{off_h(l)} + " if k == 0 else f"t[{off_t(l, k)} + "
        for j, row in enumerate(block_map(l, k, hess)):
            e = ""
            for al, v in row.items():
                t = f"M[{slots[al]}]"
                e = f"{float(v)!r} * {t}" if not e else f"fma({float(v)!r}, {t}, {e})"
            L.append(f"  {base}{j}] = (T)({'sc * (' + e + ')' if e else '0.0'});")
    return L


def gen_coefT(n):
    """Transpose of the harmonic (k = 0) map of order n: M[slot] = sum over the
    block's coefficient cotangents h of literal * h."""
    slots = monomials(n)
    rows = block_map(n, 0, False)
    L = []
    for i, al in enumerate(slots):
        e = ""
        for j, row in enumerate(rows):
            if al in row:
                t = f"h[{off_h(n) + j}]"
                e = f"{float(row[al])!r} * {t}" if not e else f"fma({float(row[al])!r}, {t}, {e})"
        L.append(f"  M[{i}] = {e if e else '0.0'};")
    return L


def gen_rows_table():
    """Cotangents of the harmonic (k = 0) coefficients -> those of the weighted
    raw moments, as sparse rows over the slots: start offsets, coefficient
    indices and values (weights divided out)."""
    start, idx, val = [0], [], []
    for n in range(PMAX + 1):
        rows = block_map(n, 0, False)
        for al in monomials(n):
            for j, row in enumerate(rows):
                if al in row:
                    idx.append(off_h(n) + j)
                    val.append(float(row[al] / weight(al)))
            start.append(len(idx))
    return start, idx, val


# ------------------------------------------------------------ kernels' bodies
def yname(l, m, s):
    return f"Y{l}_{m}{'s' if s else 'c'}"


def emit_basis(L, l, rho):
    """Degree-l basis values from degrees l-1 and l-2; rho None means 1."""
    for m, s in harmonics(l):
        nm = yname(l, m, s)
        if l == 0:
            continue
        if l == 1:
            L.append(f"  const T {nm} = {'z' if m == 0 else ('y' if s else 'x')};")
        elif m == l:
            c, d = yname(l - 1, l - 1, 0), yname(l - 1, l - 1, 1)
            L.append(f"  const T {nm} = " + (f"hot_fma(x, {d}, y * {c});" if s else
                                             f"hot_fma(x, {c}, -(y * {d}));"))
        elif m == l - 1:
            L.append(f"  const T {nm} = z * {yname(l - 1, m, s)};")
        else:
            lo = yname(l - 2, m, s) if l > 2 else "T(1)"
            if rho is None:
                if l == 2:
                    L.append(f"  const T {nm} = hot_fma(z, {yname(1, 0, 0)}, {lit(-clm(l, m))});")
                else:
                    L.append(f"  const T {nm} = hot_fma({lit(-clm(l, m))}, {lo}, "
                             f"z * {yname(l - 1, m, s)});")
            else:
                if l == 2:
                    L.append(f"  const T {nm} = hot_fma({lit(-clm(l, m))}, {rho}, "
                             f"z * {yname(1, 0, 0)});")
                else:
                    L.append(f"  const T {nm} = hot_fma({lit(-clm(l, m))}, {rho} * {lo}, "
                             f"z * {yname(l - 1, m, s)});")


def emit_row(L, names, arr, off, deg, comps, tag):
    """comps sums over the degree-deg basis: names[i] = sum_m arr[off + m comps + i] Y."""
    for j, (m, s) in enumerate(harmonics(deg)):
        for i in range(comps):
            c = f"{arr}[{off + j * comps + i}]"
            if deg == 0:
                L.append(f"  const T {names[i]}{tag} = {c};")
            elif j == 0:
                L.append(f"  T {names[i]}{tag} = {c} * {yname(deg, m, s)};")
            else:
                L.append(f"  {names[i]}{tag} = hot_fma({c}, {yname(deg, m, s)}, {names[i]}{tag});")


def gen_fwd_newton(P):
    """Newtonian multipoles on the unit vector x = R u (rho = 1): with
    v_l = u^(l+2) and g_l = grad H_l(x), G = sum v g, Q = sum (v/l) g,
      a = G + x (-H_0 u^2 - 2 x.G - x.Q),  phi = R.Q + H_0 u
    (R.Q, not x.Q / u: the monopole's potential then carries one reciprocal square
    root's rounding instead of two, and no s u where s overflows)."""
    L = ["  const T s_ = hot_fma(X, X, hot_fma(Y, Y, hot_fma(Z, Z, e2)));",
         "  const T u = hot_rsq(s_);",
         "  const T x = X * u, y = Y * u, z = Z * u;",
         "  const T v0 = u * u;",
         "  const T q0 = C[0] * v0;",
         "  T Gx = T(0), Gy = T(0), Gz = T(0), Qx = T(0), Qy = T(0), Qz = T(0);"]
    for l in range(1, P + 1):
        deg = l - 1
        if deg >= 1:
            emit_basis(L, deg, None)
        emit_row(L, ["gx", "gy", "gz"], "C", off_h(l), deg, 3, f"{l}")
        L.append(f"  const T v{l} = v{l - 1} * u;")
        if l == 1:
            for d in "xyz":
                L.append(f"  G{d} = v1 * g{d}1; Q{d} = G{d};")
        else:
            L.append(f"  const T w{l} = v{l} * {lit(Fr(1, l))};")
            for d in "xyz":
                L.append(f"  G{d} = hot_fma(v{l}, g{d}{l}, G{d}); Q{d} = hot_fma(w{l}, g{d}{l}, Q{d});")
    L += ["  const T xQ = hot_fma(x, Qx, hot_fma(y, Qy, z * Qz));",
          "  const T xG = hot_fma(x, Gx, hot_fma(y, Gy, z * Gz));",
          "  const T W = hot_fma(T(-2.0), xG, -(q0 + xQ));",
          "  ax += hot_fma(x, W, Gx); ay += hot_fma(y, W, Gy); az += hot_fma(z, W, Gz);",
          "  if constexpr (POT) ph = hot_fma(X, Qx, hot_fma(Y, Qy, hot_fma(Z, Qz, hot_fma(C[0], u, ph))));"]
    return L


def emit_radial(L, K):
    """f_n = F_n / ((-1)^(n+1) (2n-1)!!), n <= K. Plummer: u^(2n+1). K1 (e2 the
    squared kernel radius): Newtonian outside; inside F_n = -(-2)^n Q^(n)(v) /
    (256 eps^(2n+1)) with Q(v) = 256 + 128 v + 96 v^2 + 80 v^3 + 385 v^4 in
    v = 1 - |R|^2 / e2 (zero beyond n = 4), selected lane by lane."""
    e = L.append
    e("  T " + ", ".join(f"f{n}" for n in range(K + 1)) + ";")
    e("  const T rho = hot_fma(x, x, hot_fma(y, y, z * z));")
    e("  {")
    e("  const T u_ = hot_rsq(K1 ? rho : rho + e2);")
    e("  const T is_ = u_ * u_;")
    e("  f0 = u_;")
    for n in range(K):
        e(f"  f{n + 1} = f{n} * is_;")
    e("  if constexpr (K1) {")
    e("  if (rho < e2) {")
    e("  const T ie_ = hot_rsq(e2), ie2_ = ie_ * ie_;")
    e("  const T v_ = (e2 - rho) * ie2_;")
    # Q^(n) 2^n / 256, the sign of F_n and its normalisation: all positive / (2n-1)!!
    polys = [[1.0, 0.5, 0.375, 0.3125, 1.50390625], [1.0, 1.5, 1.875, 12.03125],
             [3.0, 7.5, 72.1875], [15.0, 288.75], [577.5]]
    e("  T iep_ = ie_;")
    for n in range(K + 1):
        if n < 5:
            c = [Fr(x) / dfact(2 * n - 1) for x in polys[n]]
            h = lit(c[-1])
            for co in reversed(c[:-1]):
                h = f"hot_fma(v_, {h}, {lit(co)})"
            e(f"  f{n} = iep_ * {h};")
            if n < min(K, 4):
                e("  iep_ = iep_ * ie2_;")
        else:
            e(f"  f{n} = T(0);")
    e("  }")
    e("  }")
    e("  }")


def fnorm(n):
    return Fr((-1) ** (n + 1) * dfact(2 * n - 1))


def plummer_terms(l, k):
    """g_{l,k} = (Laplacian in 3+2l dimensions)^k F_l for the Plummer kernel, as
    {(i, n): c} meaning sum c e2^i F_n: L F_n = 2 (l - n) F_{n+1} - e2 F_{n+2}."""
    t = {(0, l): Fr(1)}
    for _ in range(k):
        r = {}
        for (i, n), c in t.items():
            if l != n:
                r[(i, n + 1)] = r.get((i, n + 1), Fr(0)) + 2 * (l - n) * c
            r[(i + 1, n + 2)] = r.get((i + 1, n + 2), Fr(0)) - c
        t = r
    return t


def general_terms(l, k):
    """The same for any radial function, {(j, n): c}: sum c rho^j F_n."""
    return {(j, l + k + j): Fr(comb(k, j) * dfact(2 * l + 2 * k + 1), dfact(2 * l + 2 * j + 1))
            for j in range(k + 1)}


def emit_g(L, lmax_of, P):
    """gh{l}_{k} = g_{l,k} / norm(l) for every k >= 1 and l <= lmax_of(k)."""
    kmax = P // 2
    if kmax < 1:
        return
    L.append("  T " + ", ".join(f"gh{l}_{k}" for k in range(1, kmax + 1)
                                for l in range(lmax_of(k) + 1)) + ";")
    for k1 in (False, True):
        L.append("  if constexpr (K1) {" if k1 else "  if constexpr (!K1) {")
        var = "rho" if k1 else "e2"
        # finite, so that it leaves an f_n that has vanished at zero
        L.append(f"  const T vf_ = {var} < T(1e38) ? {var} : T(1e38);")
        var = "vf_"
        for k in range(1, kmax + 1):
            for l in range(lmax_of(k) + 1):
                terms = general_terms(l, k) if k1 else plummer_terms(l, k)
                by = {}
                for (i, n), c in terms.items():
                    by.setdefault(i, []).append((n, c * fnorm(n) / norm(l)))
                # Horner in e2 (or rho), each power's coefficient one F_n term
                e = None
                for i in range(max(by), -1, -1):
                    s = None
                    for n, c in by.get(i, []):
                        s = f"{lit(c)} * f{n}" if s is None else f"hot_fma({lit(c)}, f{n}, {s})"
                    if e is None:
                        e = s
                    else:
                        e = f"hot_fma({var}, {e}, {s})" if s else f"{var} * ({e})"
                L.append(f"  gh{l}_{k} = {e};")
        L.append("  }")


def blocks(P):
    """(l, k) of every block, by degree."""
    return [(l, k) for l in range(P + 1) for k in range((P - l) // 2 + 1)]


def gen_fwd_full(P, ks=None):
    """Any softening: every (l, k) block with its own radial functions.
    a = G + R w, G = sum g_{l,k} grad H, w = R . sum (-(2l+1)/l) g_{l+1,k} grad H
    minus the l = 0 terms; phi = R . sum (g/l) grad H + sum_k g_{0,k} H_{0,k}.
    ks selects blocks by k: None all, 0 the harmonic part, 1 the trace part."""
    def want(k):
        return ks is None or (k > 0) == (ks > 0)

    L = ["  const T x = X, y = Y, z = Z;"]
    emit_radial(L, P + 1)
    if ks != 0:
        emit_g(L, lambda k: P - 2 * k + 1, P)
    L.append("  T Gx = T(0), Gy = T(0), Gz = T(0), Qx = T(0), Qy = T(0), Qz = T(0), "
             "Px = T(0), Py = T(0), Pz = T(0);")

    def g(l, k):
        return f"f{l}" if k == 0 else f"gh{l}_{k}"

    L.append("  T w0 = C[0] * f1, p0 = C[0] * f0;" if want(0) else "  T w0 = T(0), p0 = T(0);")
    for k in range(1, P // 2 + 1):
        if want(k):
            L.append(f"  w0 = hot_fma(D[{off_t(0, k)}], {g(1, k)}, w0); "
                     f"p0 = hot_fma(D[{off_t(0, k)}], {g(0, k)}, p0);")
    for l in range(1, P + 1):
        deg = l - 1
        kl = [k for k in range((P - l) // 2 + 1) if want(k)]
        if not kl:
            continue
        if deg >= 1:
            emit_basis(L, deg, "rho")
        for k in kl:
            arr, off = ("C", off_h(l)) if k == 0 else ("D", off_t(l, k))
            emit_row(L, ["gx", "gy", "gz"], arr, off, deg, 3, f"{l}_{k}")
            L.append(f"  const T m{l}_{k} = {lit(Fr(-(2 * l + 1), l))} * {g(l + 1, k)};")
            for d in "xyz":
                L.append(f"  G{d} = hot_fma({g(l, k)}, g{d}{l}_{k}, G{d}); "
                         f"Q{d} = hot_fma(m{l}_{k}, g{d}{l}_{k}, Q{d});")
            L.append("  if constexpr (POT) {")
            L.append(f"  const T r{l}_{k} = {lit(Fr(1, l))} * {g(l, k)};")
            for d in "xyz":
                L.append(f"  P{d} = hot_fma(r{l}_{k}, g{d}{l}_{k}, P{d});")
            L.append("  }")
    L += ["  const T W = hot_fma(x, Qx, hot_fma(y, Qy, hot_fma(z, Qz, -w0)));",
          "  ax += hot_fma(x, W, Gx); ay += hot_fma(y, W, Gy); az += hot_fma(z, W, Gz);",
          "  if constexpr (POT) ph += hot_fma(x, Px, hot_fma(y, Py, hot_fma(z, Pz, p0)));"]
    return L


HN = ["xx", "xy", "xz", "yy", "yz"]


def sink_finish(L, first):
    """g from the sums over l >= 2 of v A, v/(l-1) A, v/l A (A the Hessian of H)
    and the low degrees. With c = -(2l+1)/(l-1) = -2 - 3/(l-1):
      gradient factor  c            (A x = (l-1) grad H)
      H factor         c / l = 1/l - 3/(l-1)
      second factor    -c (2l+3) / l = 4 - 3/l + 15/(l-1)."""
    for a in "012":
        L.append(f"  const T A{a}zz = -(A{a}xx + A{a}yy);")
        L.append(f"  const T V{a}x = hot_fma(A{a}xx, x, hot_fma(A{a}xy, y, A{a}xz * z));")
        L.append(f"  const T V{a}y = hot_fma(A{a}xy, x, hot_fma(A{a}yy, y, A{a}yz * z));")
        L.append(f"  const T V{a}z = hot_fma(A{a}xz, x, hot_fma(A{a}yz, y, A{a}zz * z));")
        L.append(f"  const T S{a} = hot_fma(V{a}x, x, hot_fma(V{a}y, y, V{a}z * z));")
    L += first


def gen_sink_newton(P):
    """Hessian of the expansion times b, Newtonian multipoles on x = R u:
    with v_l = u^(l+3), A_l = Hessian of H_l(x),
      g = sum v [A b + c (x (b.A x) + (b.x) A x) + (c/l) (x.A x) b
                 - c (2l+3)/l (x.A x)(b.x) x]   (l >= 2; l = 0, 1 apart)."""
    L = ["  const T s_ = hot_fma(X, X, hot_fma(Y, Y, hot_fma(Z, Z, e2)));",
         "  const T u = hot_rsq(s_);",
         "  const T x = X * u, y = Y * u, z = Z * u;",
         "  const T v0 = (u * u) * u;",
         "  const T xb = hot_fma(x, bx, hot_fma(y, by, z * bz));",
         "  const T q0 = C[0] * v0;",
         # al: factor of b; be: factor of x
         "  T al = -q0, be = T(3.0) * (q0 * xb);"]
    if P >= 1:
        L += ["  const T v1 = v0 * u;",
              "  const T hx = C[1] * v1, hy = C[2] * v1, hz = C[3] * v1;",
              "  const T hR = hot_fma(hx, x, hot_fma(hy, y, hz * z));",
              "  const T hb = hot_fma(hx, bx, hot_fma(hy, by, hz * bz));",
              "  al = hot_fma(T(-3.0), hR, al);",
              "  be = hot_fma(T(15.0) * hR, xb, hot_fma(T(-3.0), hb, be));",
              "  const T xb3 = T(-3.0) * xb;"]
    if P >= 2:
        L.append("  T " + ", ".join(f"A{a}{h} = T(0)" for a in "012" for h in HN) + ";")
    for l in range(2, P + 1):
        deg = l - 2
        if deg >= 1:
            emit_basis(L, deg, None)
        emit_row(L, [f"h{h}" for h in HN], "C", off_hh(l), deg, 5, f"{l}")
        L.append(f"  const T v{l} = v{l - 1} * u;")
        L.append(f"  const T w{l} = v{l} * {lit(Fr(1, l))};")
        if l > 2:
            L.append(f"  const T t{l} = v{l} * {lit(Fr(1, l - 1))};")
        for h in HN:
            t = f"t{l}" if l > 2 else f"v{l}"
            L.append(f"  A0{h} = hot_fma(v{l}, h{h}{l}, A0{h}); A1{h} = hot_fma({t}, h{h}{l}, A1{h}); "
                     f"A2{h} = hot_fma(w{l}, h{h}{l}, A2{h});")
    if P >= 2:
        sink_finish(L, [
            # c A x: -2 V0 - 3 V1
            "  const T Ux = hot_fma(T(-3.0), V1x, T(-2.0) * V0x);",
            "  const T Uy = hot_fma(T(-3.0), V1y, T(-2.0) * V0y);",
            "  const T Uz = hot_fma(T(-3.0), V1z, T(-2.0) * V0z);",
            "  al += hot_fma(T(-3.0), S1, S2);",
            "  const T bU = hot_fma(bx, Ux, hot_fma(by, Uy, bz * Uz));",
            "  be = hot_fma(hot_fma(T(15.0), S1, hot_fma(T(-3.0), S2, T(4.0) * S0)), xb, be + bU);",
            "  gx = hot_fma(A0xx, bx, hot_fma(A0xy, by, hot_fma(A0xz, bz, hot_fma(xb, Ux, gx))));",
            "  gy = hot_fma(A0xy, bx, hot_fma(A0yy, by, hot_fma(A0yz, bz, hot_fma(xb, Uy, gy))));",
            "  gz = hot_fma(A0xz, bx, hot_fma(A0yz, by, hot_fma(A0zz, bz, hot_fma(xb, Uz, gz))));"])
    if P >= 1:
        L += ["  gx = hot_fma(xb3, hx, gx); gy = hot_fma(xb3, hy, gy); gz = hot_fma(xb3, hz, gz);"]
    L += ["  gx = hot_fma(al, bx, hot_fma(be, x, gx)); gy = hot_fma(al, by, hot_fma(be, y, gy)); "
          "gz = hot_fma(al, bz, hot_fma(be, z, gz));"]
    return L


def gen_sink_full(P, ks=None):
    """The same for any softening, every (l, k) block with its own radial
    functions g, g' = -(2l+1) g_{l+1,k}, g'' = (2l+1)(2l+3) g_{l+2,k}:
      g = g A b + g' (R (b.grad H) + (b.R) grad H + b H) + g'' R (b.R) H.
    ks as in gen_fwd_full."""
    def want(k):
        return ks is None or (k > 0) == (ks > 0)

    L = ["  const T x = X, y = Y, z = Z;"]
    emit_radial(L, P + 2)
    if ks != 0:
        emit_g(L, lambda k: P - 2 * k + 2, P)

    def g(l, k):
        return f"f{l}" if k == 0 else f"gh{l}_{k}"

    L += ["  const T xb = hot_fma(x, bx, hot_fma(y, by, z * bz));",
          "  T al = T(0), be = T(0);"]
    for k in range(P // 2 + 1):
        if not want(k):
            continue
        c = f"C[0]" if k == 0 else f"D[{off_th(0, k)}]"
        L.append(f"  al = hot_fma({c}, -{g(1, k)}, al); "
                 f"be = hot_fma({c} * xb, T(3.0) * {g(2, k)}, be);")
    L.append("  T Ux = T(0), Uy = T(0), Uz = T(0);")
    if P >= 1:
        for k in range((P - 1) // 2 + 1):
            if not want(k):
                continue
            arr, off = ("C", off_hh(1)) if k == 0 else ("D", off_th(1, k))
            c = [f"{arr}[{off + i}]" for i in range(3)]
            L += ["  {",
                  f"  const T r = {lit(-3)} * {g(2, k)};",
                  f"  const T hR = hot_fma({c[0]}, x, hot_fma({c[1]}, y, {c[2]} * z));",
                  f"  Ux = hot_fma(r, {c[0]}, Ux); Uy = hot_fma(r, {c[1]}, Uy); "
                  f"Uz = hot_fma(r, {c[2]}, Uz);",
                  "  al = hot_fma(r, hR, al);",
                  f"  be = hot_fma(({lit(15)} * {g(3, k)}) * hR, xb, be);",
                  "  }"]
    if P >= 2:
        L.append("  T " + ", ".join(f"A{a}{h} = T(0)" for a in "0123" for h in HN) + ";")
    for l in range(2, P + 1):
        deg = l - 2
        kl = [k for k in range((P - l) // 2 + 1) if want(k)]
        if not kl:
            continue
        if deg >= 1:
            emit_basis(L, deg, "rho")
        for k in kl:
            arr, off = ("C", off_hh(l)) if k == 0 else ("D", off_th(l, k))
            t = f"{l}_{k}"
            emit_row(L, [f"h{h}" for h in HN], arr, off, deg, 5, t)
            L.append(f"  const T m{t} = {lit(Fr(-(2 * l + 1), l - 1))} * {g(l + 1, k)};")
            L.append(f"  const T n{t} = {lit(Fr(1, l))} * m{t};")
            L.append(f"  const T o{t} = {lit(Fr((2 * l + 1) * (2 * l + 3), l * (l - 1)))} * {g(l + 2, k)};")
            for h in HN:
                L.append(f"  A0{h} = hot_fma({g(l, k)}, h{h}{t}, A0{h}); "
                         f"A1{h} = hot_fma(m{t}, h{h}{t}, A1{h}); "
                         f"A2{h} = hot_fma(n{t}, h{h}{t}, A2{h}); "
                         f"A3{h} = hot_fma(o{t}, h{h}{t}, A3{h});")
    if P >= 2:
        L += ["  const T A0zz = -(A0xx + A0yy), A1zz = -(A1xx + A1yy);",
              "  Ux += hot_fma(A1xx, x, hot_fma(A1xy, y, A1xz * z));",
              "  Uy += hot_fma(A1xy, x, hot_fma(A1yy, y, A1yz * z));",
              "  Uz += hot_fma(A1xz, x, hot_fma(A1yz, y, A1zz * z));"]
        # quadratic forms x.A x of the traceless A2, A3: monomials once
        L += ["  const T qa = hot_fma(x, x, -(z * z)), qb = T(2.0) * (x * y), qc = T(2.0) * (x * z), "
              "qd = hot_fma(y, y, -(z * z)), qe = T(2.0) * (y * z);",
              "  al += hot_fma(A2xx, qa, hot_fma(A2xy, qb, hot_fma(A2xz, qc, hot_fma(A2yy, qd, A2yz * qe))));",
              "  const T S3 = hot_fma(A3xx, qa, hot_fma(A3xy, qb, hot_fma(A3xz, qc, hot_fma(A3yy, qd, A3yz * qe))));",
              "  be = hot_fma(S3, xb, be);",
              "  gx = hot_fma(A0xx, bx, hot_fma(A0xy, by, hot_fma(A0xz, bz, gx)));",
              "  gy = hot_fma(A0xy, bx, hot_fma(A0yy, by, hot_fma(A0yz, bz, gy)));",
              "  gz = hot_fma(A0xz, bx, hot_fma(A0yz, by, hot_fma(A0zz, bz, gz)));"]
    L += ["  be += hot_fma(bx, Ux, hot_fma(by, Uy, bz * Uz));",
          "  gx = hot_fma(al, bx, hot_fma(be, x, hot_fma(xb, Ux, gx)));",
          "  gy = hot_fma(al, by, hot_fma(be, y, hot_fma(xb, Uy, gy)));",
          "  gz = hot_fma(al, bz, hot_fma(be, z, hot_fma(xb, Uz, gz)));"]
    return L


def gen_cell_newton(P):
    """Cotangents of the harmonic coefficients for one sink with cotangent b:
    row[(l, m, i)] += Y_{l-1,m}(x) u_{l,i}, u_l = v_l (b - (2 + 1/l) (x.b) x),
    row[0] -= u^2 (x.b)."""
    L = ["  const T s_ = hot_fma(X, X, hot_fma(Y, Y, hot_fma(Z, Z, e2)));",
         "  const T u = hot_rsq(s_);",
         "  const T x = X * u, y = Y * u, z = Z * u;",
         "  const T xb = hot_fma(x, bx, hot_fma(y, by, z * bz));",
         "  const T v0 = u * u;",
         "  row[0] = hot_fma(-v0, xb, row[0]);"]
    if P >= 1:
        L.append("  const T px = xb * x, py = xb * y, pz = xb * z;")
    for l in range(1, P + 1):
        deg = l - 1
        if deg >= 1:
            emit_basis(L, deg, None)
        L.append(f"  const T v{l} = v{l - 1} * u;")
        for d in "xyz":
            L.append(f"  const T u{d}{l} = v{l} * hot_fma({lit(Fr(-(2 * l + 1), l))}, p{d}, b{d});")
        for j, (m, s) in enumerate(harmonics(deg)):
            for i, d in enumerate("xyz"):
                r = f"row[{off_h(l) + 3 * j + i}]"
                L.append(f"  {r} += u{d}{l};" if deg == 0 else
                         f"  {r} = hot_fma({yname(deg, m, s)}, u{d}{l}, {r});")
    return L


def flops(kind, P, softened=False):
    """Operations of the emitted expression per sink and cell, without the
    potential (kind "field", "jacobian" or "cell"; softened: the full form under
    Plummer softening): a fused multiply-add 2, any other 1."""
    gen = {"field": gen_fwd_full if softened else gen_fwd_newton,
           "jacobian": gen_sink_full if softened else gen_sink_newton, "cell": gen_cell_newton}
    n, skip, depth = 0, 0, 0
    for line in gen[kind](P):
        for st in line.split(";"):
            t = st.strip()
            opens = t.count("{") - t.count("}")
            if not skip and t.startswith(("if constexpr (K1) {", "if constexpr (POT)")):
                if opens == 0:
                    break  # a statement of its own
                skip = depth + 1
            if not skip:
                n += 2 * t.count("hot_fma(") + t.count("hot_rsq(")
                n += sum(t.count(o) for o in (" * ", " + ", " - ", " += "))
            depth += opens
            if skip and depth < skip:
                skip = 0
    return n


def dispatch(parts, head, gen):
    parts += head
    for P in range(PMAX + 1):
        parts.append(f"  {'if' if P == 0 else '} else if'} constexpr (P == {P}) {{")
        parts += gen(P)
    parts += ["  }", "}", ""]


def main(path):
    parts = ["// Generated by gen_harmonics.py -- do not edit.", "#pragma once", "namespace hot {", ""]
    dispatch(parts, ["template <int P, typename T, bool POT>",
                     "__device__ __forceinline__ void harm_fwd_newton(T X, T Y, T Z, T e2, "
                     "const T* __restrict__ C, T& ax, T& ay, T& az, T& ph) {"], gen_fwd_newton)
    dispatch(parts, ["template <int P, typename T, bool POT, bool K1>",
                     "__device__ __forceinline__ void harm_fwd_full(T X, T Y, T Z, T e2, "
                     "const T* __restrict__ C, const T* __restrict__ D, T& ax, T& ay, T& az, "
                     "T& ph) {"], gen_fwd_full)
    # its harmonic (k = 0) and trace (k >= 1) parts apart, for callers whose
    # registers hold one part's coefficients at a time
    dispatch(parts, ["template <int P, typename T, bool POT, bool K1>",
                     "__device__ __forceinline__ void harm_fwd_full_h(T X, T Y, T Z, T e2, "
                     "const T* __restrict__ C, T& ax, T& ay, T& az, T& ph) {"],
             lambda P: gen_fwd_full(P, 0))
    dispatch(parts, ["template <int P, typename T, bool POT, bool K1>",
                     "__device__ __forceinline__ void harm_fwd_full_t(T X, T Y, T Z, T e2, "
                     "const T* __restrict__ D, T& ax, T& ay, T& az, T& ph) {"],
             lambda P: gen_fwd_full(P, 1))
    dispatch(parts, ["template <int P, typename T>",
                     "__device__ __forceinline__ void harm_sink_newton(T X, T Y, T Z, T e2, "
                     "const T* __restrict__ C, T bx, T by, T bz, T& gx, T& gy, T& gz) {"],
             gen_sink_newton)
    dispatch(parts, ["template <int P, typename T, bool K1>",
                     "__device__ __forceinline__ void harm_sink_full(T X, T Y, T Z, T e2, "
                     "const T* __restrict__ C, const T* __restrict__ D, T bx, T by, T bz, T& gx, "
                     "T& gy, T& gz) {"], gen_sink_full)
    for part, arr in enumerate("CD"):
        dispatch(parts, ["template <int P, typename T, bool K1>",
                         f"__device__ __forceinline__ void harm_sink_full_{'ht'[part]}(T X, T Y, "
                         f"T Z, T e2, const T* __restrict__ {arr}, T bx, T by, T bz, T& gx, T& gy, "
                         "T& gz) {"], lambda P, part=part: gen_sink_full(P, part))
    dispatch(parts, ["template <int P, typename T>",
                     "__device__ __forceinline__ void harm_cell_newton(T X, T Y, T Z, T e2, T bx, "
                     "T by, T bz, T* row) {"], gen_cell_newton)
    for n in range(PMAX + 1):
        parts += ["template <typename T>",
                  f"__device__ __forceinline__ void harm_grad_coef{n}(const double* M, double sc, "
                  "T* __restrict__ h, T* __restrict__ t) {"] + gen_coef(n, False) + ["}"]
        parts += ["template <typename T>",
                  f"__device__ __forceinline__ void harm_hess_coef{n}(const double* M, double sc, "
                  "T* __restrict__ h, T* __restrict__ t) {"] + gen_coef(n, True) + ["}"]
    # the transposed maps, for the host tests
    parts.append("#ifndef __HIP__")
    for n in range(PMAX + 1):
        parts += [f"inline void harm_coefT{n}(const double* h, double* M) {{"] + gen_coefT(n) + ["}"]
    parts.append("#endif")
    start, idx, val = gen_rows_table()
    parts += ["struct HarmRows {", f"  short start[{len(start)}];", f"  short idx[{len(idx)}];",
              f"  double val[{len(val)}];", "};",
              "constexpr HarmRows kHarmRows = {",
              "  {" + ", ".join(map(str, start)) + "},", "  {" + ", ".join(map(str, idx)) + "},",
              "  {" + ", ".join(map(repr, val)) + "}};"]
    parts += ["", "}  // namespace hot"]
    os.makedirs(os.path.dirname(path), exist_ok=True)
    tmp = path + ".tmp"
    with open(tmp, "w") as f:
        f.write("\n".join(parts) + "\n")
    os.replace(tmp, path)


if __name__ == "__main__":
    main(sys.argv[1] if len(sys.argv) > 1 else
         os.path.join(os.path.dirname(os.path.abspath(__file__)), "generated", "harmonics.h"))
