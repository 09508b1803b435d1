"""Build-time generator of the constant tables and unrolled SH-product code.

Writes ``generated/shv_constants.h`` and ``generated/shv_gaunt.h`` for the HIP
library.  Everything here is derived from closed forms:

  * real SH normalisation K_l^m = sqrt((2l+1)/(4 pi) (l-m)!/(l+m)!) and a
    scaled associated-Legendre recurrence in z (index i = l*l + l + m, the
    linearisation of Sec. 3.2);
  * triple-product coefficients C_ijk = integral y_i y_j y_k (Eq. 7) from the
    Wigner 3j symbols (Racah's formula, exact rational arithmetic) and the
    unitary map between complex and real harmonics;
  * clamped-cosine Funk-Hecke eigenvalues A_l (Eqs. 10-11) from the
    Ramamoorthi-Hanrahan closed form;
  * log-cap zonal constants 2 pi / (2l + 1) (Eq. 13 projected about z).

Basis convention: real, orthonormal, no Condon-Shortley phase, y_lm ~ cos(m phi)
for m > 0 and sin(|m| phi) for m < 0.

The generated SH-product code is straight-line: registers cannot be indexed by
data on the GPU, so each sparse contraction is unrolled at compile time with
its coefficients as literals.

Run:  python gen_tables.py <out_dir>
"""
from __future__ import annotations

import math

import numpy as np
import os
import sys
from fractions import Fraction

MAX_BANDS = 8
PI = math.pi


# ----------------------------------------------------------------- Wigner 3j

def _f(n):
    return math.factorial(n)


def wigner3j(j1, j2, j3, m1, m2, m3) -> float:
    if m1 + m2 + m3 != 0:
        return 0.0
    if j3 < abs(j1 - j2) or j3 > j1 + j2:
        return 0.0
    if abs(m1) > j1 or abs(m2) > j2 or abs(m3) > j3:
        return 0.0
    tri = Fraction(_f(j1 + j2 - j3) * _f(j1 - j2 + j3) * _f(-j1 + j2 + j3), _f(j1 + j2 + j3 + 1))
    pre = tri * _f(j1 + m1) * _f(j1 - m1) * _f(j2 + m2) * _f(j2 - m2) * _f(j3 + m3) * _f(j3 - m3)
    s = Fraction(0)
    kmin = max(0, j2 - j3 - m1, j1 - j3 + m2)
    kmax = min(j1 + j2 - j3, j1 - m1, j2 + m2)
    for k in range(kmin, kmax + 1):
        den = (_f(k) * _f(j3 - j2 + k + m1) * _f(j3 - j1 + k - m2) * _f(j1 + j2 - j3 - k)
               * _f(j1 - k - m1) * _f(j2 - k + m2))
        s += Fraction((-1) ** k, den)
    sign = -1 if (j1 - j2 - m3) % 2 else 1
    # value = sign * sqrt(pre) * s, evaluated as sqrt(pre * s^2) with s's sign
    mag = math.sqrt(float(pre * s * s))
    return sign * (1 if s >= 0 else -1) * mag


def complex_gaunt(l1, m1, l2, m2, l3, m3) -> float:
    """integral Y_l1^m1 Y_l2^m2 Y_l3^m3 (no conjugation, Condon-Shortley phase)."""
    if m1 + m2 + m3 != 0 or (l1 + l2 + l3) % 2:
        return 0.0
    w0 = wigner3j(l1, l2, l3, 0, 0, 0)
    if w0 == 0.0:
        return 0.0
    return math.sqrt((2 * l1 + 1) * (2 * l2 + 1) * (2 * l3 + 1) / (4 * PI)) * w0 * wigner3j(l1, l2, l3, m1, m2, m3)


def real_to_complex(l, m):
    """Coefficients u with y_lm = sum_m' u[m'] Y_l^m' (complex dict)."""
    if m == 0:
        return {0: 1.0 + 0j}
    a = abs(m)
    s = (-1) ** a
    if m > 0:
        return {a: s / math.sqrt(2) + 0j, -a: 1 / math.sqrt(2) + 0j}
    return {a: -1j * s / math.sqrt(2), -a: 1j / math.sqrt(2)}


def lm(i):
    l = math.isqrt(i)
    return l, i - l * l - l


def real_gaunt(n_bands):
    """Dict (i, j, k) -> C_ijk (nonzero entries only) for i, j, k < n^2."""
    N = n_bands * n_bands
    out = {}
    for i in range(N):
        li, mi = lm(i)
        ui = real_to_complex(li, mi)
        for j in range(i, N):
            lj, mj = lm(j)
            uj = real_to_complex(lj, mj)
            for k in range(j, N):
                lk, mk = lm(k)
                if (li + lj + lk) % 2 or lk > li + lj or lk < abs(li - lj):
                    continue
                uk = real_to_complex(lk, mk)
                acc = 0j
                for a, ca in ui.items():
                    for b, cb in uj.items():
                        c = -a - b
                        if c in uk:
                            acc += ca * cb * uk[c] * complex_gaunt(li, a, lj, b, lk, c)
                assert abs(acc.imag) < 1e-12, (i, j, k, acc)
                if abs(acc.real) > 1e-13:
                    for p in {(i, j, k), (i, k, j), (j, i, k), (j, k, i), (k, i, j), (k, j, i)}:
                        out[p] = acc.real
    return out


# ----------------------------------------------------------------- basis constants

def dfact(n):
    r = 1
    while n > 1:
        r *= n
        n -= 2
    return r


def norm_c(l, m):
    k = math.sqrt((2 * l + 1) / (4 * PI) * _f(l - m) / _f(l + m))
    return k if m == 0 else math.sqrt(2.0) * k


def recurrence_constants():
    """r_lm = Q_l^m(z) / mu_lm with Q_l^m = d^m P_l / dz^m:
         r_mm = 1, r_{m+1,m} = z, r_lm = z r_{l-1,m} + gamma_lm r_{l-2,m};
       y_lm = lam_lm r_lm T_m(x, y) with T_m = Re/Im (x + i y)^|m|;
       d r_lm / dz = rho_lm r_{l,m+1}."""
    mu = {}
    for m in range(MAX_BANDS + 1):
        mu[(m, m)] = Fraction(dfact(2 * m - 1))
        for l in range(m + 1, MAX_BANDS + 1):
            mu[(l, m)] = mu[(l - 1, m)] * Fraction(2 * l - 1, l - m)
    gamma = [[0.0] * MAX_BANDS for _ in range(MAX_BANDS)]
    lam = [[0.0] * MAX_BANDS for _ in range(MAX_BANDS)]
    rho = [[0.0] * MAX_BANDS for _ in range(MAX_BANDS)]
    for l in range(MAX_BANDS):
        for m in range(l + 1):
            if l >= m + 2:
                gamma[l][m] = float(-Fraction(l + m - 1, l - m) * mu[(l - 2, m)] / mu[(l, m)])
            lam[l][m] = norm_c(l, m) * float(mu[(l, m)])
            rho[l][m] = float(mu[(l, m + 1)] / mu[(l, m)]) if m + 1 <= l else 0.0
    return gamma, lam, rho


def pair_constants():
    """The pair kernels' basis (shv_device.h).  With Q_l^m = d^m P_l / dz^m:
         p_l = P_l / its leading coefficient (m = 0),
         rho_l^m = Q_l^m / kappa, m >= 1, kappa = (2m - 1)!! where l - m is even and (2m + 1)!! where it is odd,
         so rho_m^m = 1, rho_{m+1}^m = z, and Q_l^m = Q_{l-2}^m + (2l - 1) Q_{l-1}^{m-1} has one constant, ROW;
         a_0 = 1 - t, a_l = (1 - t^2) P_l'(t) / its leading coefficient: the zonal terms, d a_l / dt = -(l + 1) p_l.
       Returns (pair, row, row_k, row_0, cap_b, leg_b): y_lm g_l = pair a_l rho_l^m T_m (at m = 0, p_l for rho),
       ROW, d rho_l^m / dz over rho_l^{m+1} (l - m even; 1 where odd) and at m = 0 d p_l / dz over rho_l^1, and the
       recurrences' a_{l+1} = t a_l - cap_b a_{l-1}, p_{l+1} = t p_l - leg_b p_{l-1}."""
    lead = lambda l, m: Fraction(_f(2 * l), 2 ** l * _f(l) * _f(l - m))  # noqa: E731
    kappa = lambda m, odd: Fraction(dfact(2 * m + 1 if odd else 2 * m - 1))  # noqa: E731
    pair = [[0.0] * MAX_BANDS for _ in range(MAX_BANDS)]
    row = [[0.0] * MAX_BANDS for _ in range(MAX_BANDS)]
    for l in range(MAX_BANDS):
        # g_l = -2 pi u, -2 pi (1 - t^2) P_l'(t) / (l (l + 1))
        zonal = -2 * PI if l == 0 else -2 * PI * float(lead(l, 1) / (l * (l + 1)))
        for m in range(l + 1):
            odd = (l - m) % 2
            pair[l][m] = zonal * norm_c(l, m) * float(kappa(m, odd) if m else lead(l, 0))
            if l >= m + 2 and m >= 1:
                below = kappa(m - 1, odd) if m > 1 else lead(l - 1, 0)
                row[l][m] = float((2 * l - 1) * below / kappa(m, odd))
    row_k = [float((2 * m + 1) * (2 * m + 3)) for m in range(MAX_BANDS)]
    row_0 = [0.0] + [float(kappa(1, (l - 1) % 2) / lead(l, 0)) for l in range(1, MAX_BANDS)]
    cap_b = [0.0] + [(l - 1) * (l + 1) / ((2 * l - 1) * (2 * l + 1)) for l in range(1, MAX_BANDS)]
    leg_b = [l * l / ((2 * l - 1) * (2 * l + 1)) for l in range(MAX_BANDS)]
    return pair, row, row_k, row_0, cap_b, leg_b


def clamped_cosine(l):
    if l == 0:
        return PI
    if l == 1:
        return 2 * PI / 3
    if l % 2:
        return 0.0
    return 2 * PI * (-1) ** (l // 2 - 1) / ((l + 2) * (l - 1)) * _f(l) / (2 ** l * _f(l // 2) ** 2)


N_GROUPS = 4


def parity_groups(n, adjoint, ng=N_GROUPS):
    """Output groups of a squaring (one per wave of the four-wave kernels).
    Cost of a group: forward = its FMAs plus the distinct products e_j e_k it
    needs; adjoint = its terms plus twice the distinct symmetric products
    ob_i e_k it needs.  Start from the classes (l odd, m < 0): the selection
    rules of the real Gaunt coefficients make the products a class needs
    largely shared within it.  Then take best-improvement single moves while
    they lower the largest group cost.  Deterministic."""
    import collections
    N = n * n
    C = real_gaunt(n)
    ft = {i: [] for i in range(N)}
    at = {m: set() for m in range(N)}
    for (i, j, k) in C:
        if j <= k:
            ft[i].append((j, k))
        at[j].add((i, k) if i <= k else (k, i))
    at = {m: sorted(v) for m, v in at.items()}
    grp = []
    for i in range(N):
        l, m = lm(i)
        grp.append((2 * (l % 2) + (1 if m < 0 else 0)) % ng)
    fc = [collections.Counter() for _ in range(ng)]
    ac = [collections.Counter() for _ in range(ng)]
    fterm, aterm = [0] * ng, [0] * ng

    def add(i, g, sgn):
        if sgn > 0:
            fc[g].update(ft[i])
            ac[g].update(at[i])
        else:
            fc[g].subtract(ft[i])
            ac[g].subtract(at[i])
            fc[g] += collections.Counter()
            ac[g] += collections.Counter()
        fterm[g] += sgn * len(ft[i])
        aterm[g] += sgn * len(at[i])

    for i in range(N):
        add(i, grp[i], 1)

    def score():
        if adjoint:
            return max(aterm[g] + 2 * len(ac[g]) for g in range(ng))
        return max(fterm[g] + len(fc[g]) for g in range(ng))

    cur = score()
    while True:
        best = None
        for i in range(N):
            a = grp[i]
            for b in range(ng):
                if b == a:
                    continue
                add(i, a, -1)
                add(i, b, 1)
                s = score()
                add(i, b, -1)
                add(i, a, 1)
                if s < cur and (best is None or s < best[0]):
                    best = (s, i, b)
        if best is None:
            break
        cur, i, b = best
        add(i, grp[i], -1)
        add(i, b, 1)
        grp[i] = b
    return [sorted(i for i in range(N) if grp[i] == g) for g in range(ng)]


def forward_groups(n, ng=N_GROUPS):
    return order_groups(n, ng) if n >= LAT_MIN_BANDS else parity_groups(n, False, ng)


def adjoint_groups(n, ng=N_GROUPS):
    """Also the canonical grouping of the backward's sums."""
    return order_groups(n, ng) if n >= LAT_MIN_BANDS else parity_groups(n, True, ng)


# ------------------------------------------------ products through latitudes

LAT_MIN_BANDS = 6  # products through latitudes from this band count up (see shv_lat.h)


def order_groups(n, ng=N_GROUPS):
    """Output groups of a product through latitudes: whole orders |m|, since
    an order's coefficients share its Fourier product.  Cost of order m: its
    complex terms at every latitude plus its transposed transform; the orders
    are assigned in decreasing cost to the least loaded group."""
    cost = {m: (2 * n - 1 - m) * 4 * ((3 * n - 1) // 2) + 5 * 2 * (n - m) for m in range(1, n)}
    cost[0] = (2 * n - 1) * 2 * ((3 * n - 1) // 2) + 5 * n
    load, grp = [0] * ng, {}
    for m in sorted(cost, key=lambda m: -cost[m]):
        g = load.index(min(load))
        grp[m] = g
        load[g] += cost[m]
    return [sorted(i for i in range(n * n) if grp[abs(lm(i)[1])] == g) for g in range(ng)]


def lat_row(n, z, scale):
    """Entries (m, l), m-major, of scale sqrt(4 pi) N_lm P_l^m(z), N_lm P_l^m
    being y_lm without its azimuth function (and without the sqrt 2 that has
    for m > 0), padded to a multiple of four."""
    out = []
    r = math.sqrt(1 - z * z)
    for m in range(n):
        p = math.sqrt((2 * m + 1) * math.prod((2 * i - 1) / (2 * i) for i in range(1, m + 1))) * r ** m
        prev, cur = 0.0, p
        for l in range(m, n):
            if l > m:
                a = math.sqrt((4 * l * l - 1) / (l * l - m * m))
                b = math.sqrt(((l - 1) ** 2 - m * m) / (4 * (l - 1) ** 2 - 1)) if l > m + 1 else 0.0
                prev, cur = cur, a * (z * cur - b * prev)
            out.append(scale * cur)
    return out + [0.0] * (-len(out) % 4)


def lat_rows(n):
    """The Gauss-Legendre latitudes z > 0 of the rule that integrates the
    triple products of n bands exactly (degree 3 n - 3), and z = 0 where the
    rule has it: one lat_row each, scaled by w^(1/3).  The transform of each
    factor and the transposed transform carry w^(1/3) each, so a product
    carries the weight w = 2 (w / 2): the projection of twice the product."""
    zs, ws = np.polynomial.legendre.leggauss((3 * n - 3) // 2 + 1)
    pairs = [lat_row(n, z, w ** (1 / 3)) for z, w in zip(zs, ws) if z > 1e-9]
    eq = [lat_row(n, 0.0, w ** (1 / 3)) for z, w in zip(zs, ws) if abs(z) <= 1e-9]
    return pairs, eq


def emit_lat(L):
    lamb = pair_constants()[0]
    for name, f in (("SHV_LAT_LAM", lambda m: (1.0 if m == 0 else math.sqrt(0.5)) / math.sqrt(4 * PI)),
                    ("SHV_LAT_LAMI", lambda m: 1.0 if m == 0 else math.sqrt(2.0))):
        L.append(f"// PAIR[l][m] times {'the scale of a coefficient' if name.endswith('M') else '1 / (sqrt(4 pi) scale)'}.")
        L.append(f"static constexpr float {name}[{MAX_BANDS}][{MAX_BANDS}] = {{")
        for l in range(MAX_BANDS):
            L.append("  {" + ", ".join(flit(lamb[l][m] * f(m)) for m in range(MAX_BANDS)) + "},")
        L.append("};")
    L.append("static constexpr float SHV_LAT_INV[2] = {" + flit(math.sqrt(4 * PI)) + ", " + flit(math.sqrt(8 * PI))
             + "};  // 1 / scale, m = 0 and m != 0")
    L.append("static constexpr float SHV_LAT_SCALE[2] = {" + flit(1 / math.sqrt(4 * PI)) + ", "
             + flit(1 / math.sqrt(8 * PI)) + "};")
    L.append("// Products through latitudes (shv_lat.h): the rows of the pairs +-z, then of the equator.")
    for n in range(LAT_MIN_BANDS, MAX_BANDS + 1):
        pairs, eq = lat_rows(n)
        vals = [v for r in pairs + eq for v in r]
        L.append(f"static constexpr int SHV_LAT_PAIRS_{n} = {len(pairs)}, SHV_LAT_EQ_{n} = {len(eq)};")
        L.append(f"static constexpr float shv_lat_rows_{n}[{len(vals)}] = {{" + ",".join(flit(v) for v in vals) + "};")
        for name, grs in (("SHV_FGRP", forward_groups(n)), ("SHV_GRP", adjoint_groups(n))):
            gid = [0] * (n * n)
            for g, members in enumerate(grs):
                for i in members:
                    gid[i] = g
            L.append(f"static constexpr unsigned char {name}_{n}[{n * n}] = {{" + ",".join(map(str, gid)) + "};")


def real_basis(d, n):
    """y_i, i < n^2, at unit directions d [..., 3], in 64 bits."""
    x, y, z = d[..., 0], d[..., 1], d[..., 2]
    cm, sm = [np.ones_like(x)], [np.zeros_like(x)]
    for m in range(1, n):
        cm.append(cm[-1] * x - sm[-1] * y)
        sm.append(sm[-1] * x + cm[m - 1] * y)
    out = [None] * (n * n)
    for m in range(n):
        norm = math.sqrt((2 * m + 1) / (4 * PI) * math.prod((2 * i - 1) / (2 * i) for i in range(1, m + 1)))
        prev, cur = 0.0, np.full_like(z, norm * (math.sqrt(2) if m else 1.0))
        for l in range(m, n):
            if l > m:
                a = math.sqrt((4 * l * l - 1) / (l * l - m * m))
                b = math.sqrt(((l - 1) ** 2 - m * m) / (4 * (l - 1) ** 2 - 1)) if l > m + 1 else 0.0
                prev, cur = cur, a * (z * cur - b * prev)
            out[l * l + l + m] = cur * cm[m]
            if m:
                out[l * l + l - m] = cur * sm[m]
    return np.stack(out, -1)


def quarter_turn():
    """K: the rotation by 90 degrees about x (y to z) on real SH vectors,
    (K f)(w) = f(K^-1 w), by exact quadrature.  With Z(a) the rotation about z,
    the rotation about y is K^-1 Z(a) K."""
    n = MAX_BANDS
    zs, ws = np.polynomial.legendre.leggauss(2 * n)
    ph = np.arange(4 * n) * 2 * PI / (4 * n)
    st = np.sqrt(1 - zs * zs)
    d = np.stack([st[:, None] * np.cos(ph), st[:, None] * np.sin(ph), zs[:, None] + 0 * ph], -1).reshape(-1, 3)
    w = np.repeat(ws * 2 * PI / (4 * n), 4 * n)
    K = (real_basis(d, n) * w[:, None]).T @ real_basis(np.stack([d[:, 0], d[:, 2], -d[:, 1]], -1), n)
    K[np.abs(K) < 1e-12] = 0.0
    return K


def z_turn(a, derivative=False):
    """The rotation by a about z on real SH vectors, or its derivative at 0."""
    N = MAX_BANDS ** 2
    Z = np.zeros((N, N))
    for i in range(N):
        l, m = lm(i)
        j = l * l + l - m
        if derivative:
            Z[i, j] -= m
        else:
            Z[i, i] = math.cos(m * a)
            if m:
                Z[i, j] = -math.sin(m * a)
    return Z


def turn_groups(n, ng=N_GROUPS):
    """Bands l and orders m dealt to the waves of the product chain: the bands
    for the rotations (block-diagonal in l), the orders for the products with a
    zonal function (block-diagonal in m), each to the least loaded wave."""
    out = []
    for cost in ({l: 2 * l + 1 for l in range(n)}, {m: (n - m) * (2 if m else 1) for m in range(n)}):
        load, grp = [0] * ng, {}
        for k in sorted(cost, key=lambda k: -cost[k]):
            g = load.index(min(load))
            grp[k] = g
            load[g] += cost[k]
        out.append([grp[k] for k in range(n)])
    return out


def emit_turns(L):
    """Rotations and rotation cotangents band by band, on coefficients scaled
    as in shv_lat.h (entry m + l of band l), and the product chain's tables."""
    K = quarter_turn()
    Lz = z_turn(0.0, True)
    Ly = K.T @ Lz @ K
    A = K.T @ z_turn(-PI / 2) @ K   # takes x to z
    Lx = A.T @ Lz @ A
    s = np.array([1.0 if lm(i)[1] == 0 else math.sqrt(0.5) for i in range(MAX_BANDS ** 2)])
    L.append("// Rotations of SH vectors band by band (shv_prod_impl.h).")
    for l in range(MAX_BANDS):
        b = slice(l * l, (l + 1) ** 2)
        for name, M in (("turn", K[b, b]), ("unturn", K[b, b].T)):
            L.append(f"__device__ __forceinline__ void shv_{name}_l{l}(const float* v, float* o) {{")
            for i in range(2 * l + 1):
                e = None
                for j in range(2 * l + 1):
                    c = M[i, j] * s[b][i] / s[b][j]
                    if abs(c) < 1e-12:
                        continue
                    t = f"v[{j}]" if abs(c - 1) < 1e-12 else f"{flit(c)} * v[{j}]"
                    e = t if e is None else f"fmaf({flit(c)}, v[{j}], {e})"
                L.append(f"  o[{i}] = {e};")
            L.append("}")
        # gx = -<Ly v, t>, gy = <Lx v, t>, with 1 / scale^2 (up to 4 pi): the
        # generators are antisymmetric, so each pair of entries is one term
        L.append(f"__device__ __forceinline__ void shv_torque_l{l}(const float* v, const float* t, float& gx, float& gy) {{")
        for var, M in (("gx", -Ly[b, b]), ("gy", Lx[b, b])):
            for i in range(2 * l + 1):
                for j in range(i):
                    c = M[i, j] / (s[b][i] * s[b][j])
                    if abs(c) > 1e-12:
                        L.append(f"  {var} = fmaf({flit(c)}, fmaf(v[{j}], t[{i}], -(v[{i}] * t[{j}])), {var});")
        L.append("}")
    L.append("// A zonal function at the latitudes of shv_lat_rows: twice (2 l + 1) / (4 pi) P_l(z) w^(1/3)")
    L.append("// (the sum and difference of the values at z and -z), once at the equator; and the waves'")
    L.append("// bands and orders.")
    for n in range(LAT_MIN_BANDS, MAX_BANDS + 1):
        zs, ws = np.polynomial.legendre.leggauss((3 * n - 3) // 2 + 1)
        vals = []
        for z, w in [(z, w) for z, w in zip(zs, ws) if z > 1e-9] + [(z, w) for z, w in zip(zs, ws) if abs(z) <= 1e-9]:
            z = z if z > 1e-9 else 0.0
            for l in range(n):
                c = np.zeros(l + 1)
                c[l] = 1.0
                vals.append((2.0 if z else 1.0) * (2 * l + 1) / (4 * PI) * np.polynomial.legendre.legval(z, c) * w ** (1 / 3))
        L.append(f"static constexpr float shv_zonal_rows_{n}[{len(vals)}] = {{" + ",".join(flit(v) for v in vals) + "};")
        lg, mg = turn_groups(n)
        L.append(f"static constexpr unsigned char SHV_TURN_L_{n}[{n}] = {{" + ",".join(map(str, lg)) + "};")
        L.append(f"static constexpr unsigned char SHV_TURN_M_{n}[{n}] = {{" + ",".join(map(str, mg)) + "};")


def emit_quad(L):
    """The product rule of degree 8 n - 1: 4 n Gauss-Legendre latitudes, as
    the rows and weights of the pairs +-z, and 8 n azimuths (j + 1/2) 2 pi / 8 n,
    as the cosines and sines of m phi_j in the first quarter."""
    L.append("// Quadrature of the projected exponential (shv_quad_impl.h).")
    lamb = pair_constants()[0]
    for n in range(1, MAX_BANDS + 1):
        zs, ws = np.polynomial.legendre.leggauss(4 * n)
        up = [(z, w) for z, w in zip(zs, ws) if z > 0]
        rows = [v for z, _ in up for v in lat_row(n, z, 1.0)]
        L.append(f"static constexpr float shv_quad_rows_{n}[{len(rows)}] = {{" + ",".join(flit(v) for v in rows) + "};")
        # the weight of each of the latitude's azimuths
        L.append(f"static constexpr float shv_quad_w_{n}[{len(up)}] = {{"
                 + ",".join(flit(w * 2 * PI / (8 * n)) for _, w in up) + "};")
        for name, f in (("cos", math.cos), ("sin", math.sin)):
            L.append(f"static constexpr float shv_quad_{name}_{n}[{2 * n}][{n}] = {{" + ",".join(
                "{" + ",".join(flit(f(m * (j + 0.5) * 2 * PI / (8 * n))) for m in range(n)) + "}"
                for j in range(2 * n)) + "};")
    for name, f in (("norm", lambda l, m: (1.0 if m == 0 else math.sqrt(2.0)) / math.sqrt(4 * PI)),
                    ("lam", lambda l, m: lamb[l][abs(m)])):
        L.append(f"// {'y_lm over its row entry' if name == 'norm' else 'PAIR[l][|m|]'}, by coefficient index.")
        L.append(f"static constexpr float shv_coef_{name}[{MAX_BANDS ** 2}] = {{"
                 + ",".join(flit(f(*lm(i))) for i in range(MAX_BANDS ** 2)) + "};")


# ----------------------------------------------------------------- emission

def float32_rest(x: float) -> float:
    """What the nearest float32 leaves of x."""
    import struct
    return x - struct.unpack("f", struct.pack("f", x))[0]


def flit(x: float) -> str:
    """float literal that round-trips the nearest float32."""
    import struct
    f = struct.unpack("f", struct.pack("f", x))[0]
    s = repr(f)
    if "e" not in s and "." not in s:
        s += ".0"
    return s + "f"


def emit_constants(path):
    gamma, lam, rho = recurrence_constants()
    lines = ["// Generated by gen_tables.py: SH recurrence and transfer constants.",
             "#pragma once", "", f"#define SHV_MAX_BANDS {MAX_BANDS}", ""]

    def table2(name, t):
        lines.append(f"static constexpr float {name}[{MAX_BANDS}][{MAX_BANDS}] = {{")
        for row in t:
            lines.append("  {" + ", ".join(flit(v) for v in row) + "},")
        lines.append("};")

    table2("SHV_GAMMA", gamma)
    table2("SHV_LAMBDA", lam)
    table2("SHV_RHO", rho)
    pair, row, row_k, row_0, cap_b, leg_b = pair_constants()
    table2("SHV_PAIR", pair)
    table2("SHV_PAIR_LO", [[float32_rest(v) for v in r] for r in pair])
    table2("SHV_ROW", row)
    for name, t in (("SHV_ROW_K", row_k), ("SHV_ROW_0", row_0), ("SHV_CAP_B", cap_b), ("SHV_LEG_B", leg_b)):
        lines.append(f"static constexpr float {name}[{MAX_BANDS}] = {{" + ", ".join(flit(v) for v in t) + "};")
    lines.append(f"static constexpr float SHV_AHAT[{MAX_BANDS}] = {{"
                 + ", ".join(flit(clamped_cosine(l)) for l in range(MAX_BANDS)) + "};")
    # log-cap zonal: g_l(t) = -eps * 2 pi/(2l+1) * (P_{l-1}(t) - P_{l+1}(t))
    lines.append(f"static constexpr float SHV_CAPK[{MAX_BANDS}] = {{"
                 + ", ".join(flit(-2 * PI / (2 * l + 1)) for l in range(MAX_BANDS)) + "};")
    # Bonnet: P_{l+1} = (2l+1)/(l+1) t P_l - l/(l+1) P_{l-1}
    lines.append(f"static constexpr float SHV_BONNET_A[{MAX_BANDS + 1}] = {{"
                 + ", ".join(flit((2 * l + 1) / (l + 1)) for l in range(MAX_BANDS + 1)) + "};")
    lines.append(f"static constexpr float SHV_BONNET_B[{MAX_BANDS + 1}] = {{"
                 + ", ".join(flit(l / (l + 1)) for l in range(MAX_BANDS + 1)) + "};")
    lines.append("static constexpr float SHV_SQRT_4PI = " + flit(math.sqrt(4 * PI)) + ";")
    lines.append("static constexpr float SHV_INV_SQRT_4PI = " + flit(1 / math.sqrt(4 * PI)) + ";")
    lines.append("static constexpr float SHV_INV_8PI = " + flit(1 / (8 * PI)) + ";")
    lines.append("static constexpr float SHV_INV_4PI = " + flit(1 / (4 * PI)) + ";")
    lines.append("static constexpr float SHV_TWO_PI = " + flit(2 * PI) + ";")
    open(path, "w").write("\n".join(lines) + "\n")


def transfer_support(n):
    """Coefficient indices where the clamped-cosine transfer can be nonzero."""
    return [i for i in range(n * n) if clamped_cosine(lm(i)[0]) != 0.0]


def mtable(N, C):
    """Sparse table grouped by (j, k) for building M(L)_jk = sum_i L_i C_ijk."""
    rows = [[] for _ in range(N * N)]
    for (i, j, k), c in C.items():
        rows[j * N + k].append((i, c))
    ptr, ent_i, ent_c = [0], [], []
    for r in rows:
        for i, c in sorted(r):
            ent_i.append(i)
            ent_c.append(c)
        ptr.append(len(ent_i))
    return ptr, ent_i, ent_c


def emit_gaunt(path):
    L = ["// Generated by gen_tables.py: unrolled sparse SH triple products.",
         "// C_ijk = integral y_i y_j y_k from Wigner 3j symbols; straight-line code",
         "// because GPU registers cannot be indexed by data.",
         "#pragma once", ""]
    tables = []
    for n in range(1, MAX_BANDS + 1):
        N = n * n
        C = real_gaunt(n)
        nnz = len(C)
        sym = sorted((i, j, k) for (i, j, k) in C if j <= k)
        L.append(f"// n = {n}: {nnz} nonzero C_ijk, {len(sym)} with j <= k")
        L.append(f"#define SHV_GAUNT_NNZ_{n} {nnz}")
        tables.append((n, *mtable(N, C)))
        if n >= LAT_MIN_BANDS:
            continue

        # o = e * e (symmetric squaring)
        L.append(f"__device__ __forceinline__ void shv_square_{n}(const float* __restrict__ e, float* __restrict__ o) {{")
        touched = set()
        pairs = {}
        for (i, j, k) in sym:
            pairs.setdefault((j, k), []).append(i)
        for (j, k) in sorted(pairs):
            L.append(f"  {{ const float t = e[{j}] * e[{k}];")
            for i in pairs[(j, k)]:
                c = C[(i, j, k)] * (2.0 if j < k else 1.0)
                if i in touched:
                    L.append(f"    o[{i}] = fmaf({flit(c)}, t, o[{i}]);")
                else:
                    L.append(f"    o[{i}] = {flit(c)} * t;")
                    touched.add(i)
            L.append("  }")
        for i in range(N):
            if i not in touched:
                L.append(f"  o[{i}] = 0.0f;")
        L.append("}")

        # eb = 2 * (ob * e): adjoint of o = e * e
        L.append(f"__device__ __forceinline__ void shv_square_adj_{n}(const float* __restrict__ ob, const float* __restrict__ e, float* __restrict__ eb) {{")
        touched = set()
        upairs = {}
        for (j, i, k) in C:           # eb_j += 2 C_jik ob_i e_k
            if i <= k:
                upairs.setdefault((i, k), []).append(j)
        for (i, k) in sorted(upairs):
            if i == k:
                L.append(f"  {{ const float u = ob[{i}] * e[{i}];")
            else:
                L.append(f"  {{ const float u = fmaf(ob[{i}], e[{k}], ob[{k}] * e[{i}]);")
            for j in sorted(upairs[(i, k)]):
                c = 2.0 * C[(j, i, k)]
                if j in touched:
                    L.append(f"    eb[{j}] = fmaf({flit(c)}, u, eb[{j}]);")
                else:
                    L.append(f"    eb[{j}] = {flit(c)} * u;")
                    touched.add(j)
            L.append("  }")
        for j in range(N):
            if j not in touched:
                L.append(f"  eb[{j}] = 0.0f;")
        L.append("}")

        # Per-group variants for kernels that split one receiver's squaring
        # over several waves: group g computes only its outputs, with exactly
        # the per-output term order of the full functions above.
        groups = forward_groups(n)
        agroups = adjoint_groups(n)
        for name, grs in (("SHV_FGRP", groups), ("SHV_GRP", agroups)):
            gid = [0] * N
            for g, members in enumerate(grs):
                for i in members:
                    gid[i] = g
            L.append(f"static constexpr unsigned char {name}_{n}[{N}] = {{" + ",".join(map(str, gid)) + "};")
        for g, members in enumerate(groups):
            mem = set(members)
            L.append(f"__device__ __forceinline__ void shv_square_{n}_g{g}(const float* __restrict__ e, float* __restrict__ o) {{")
            touched = set()
            for (j, k) in sorted(pairs):
                outs = [i for i in pairs[(j, k)] if i in mem]
                if not outs:
                    continue
                L.append(f"  {{ const float t = e[{j}] * e[{k}];")
                for i in outs:
                    c = C[(i, j, k)] * (2.0 if j < k else 1.0)
                    if i in touched:
                        L.append(f"    o[{i}] = fmaf({flit(c)}, t, o[{i}]);")
                    else:
                        L.append(f"    o[{i}] = {flit(c)} * t;")
                        touched.add(i)
                L.append("  }")
            for i in members:
                if i not in touched:
                    L.append(f"  o[{i}] = 0.0f;")
            L.append("}")
        for g, members in enumerate(agroups):
            mem = set(members)
            L.append(f"__device__ __forceinline__ void shv_square_adj_{n}_g{g}(const float* __restrict__ ob, const float* __restrict__ e, float* __restrict__ eb) {{")
            touched = set()
            for (i, k) in sorted(upairs):
                outs = [j for j in sorted(upairs[(i, k)]) if j in mem]
                if not outs:
                    continue
                if i == k:
                    L.append(f"  {{ const float u = ob[{i}] * e[{i}];")
                else:
                    L.append(f"  {{ const float u = fmaf(ob[{i}], e[{k}], ob[{k}] * e[{i}]);")
                for j in outs:
                    c = 2.0 * C[(j, i, k)]
                    if j in touched:
                        L.append(f"    eb[{j}] = fmaf({flit(c)}, u, eb[{j}]);")
                    else:
                        L.append(f"    eb[{j}] = {flit(c)} * u;")
                        touched.add(j)
                L.append("  }")
            for j in members:
                if j not in touched:
                    L.append(f"  eb[{j}] = 0.0f;")
            L.append("}")

        L.append("")

    L.append("// (j, k)-grouped sparse C for building M(L); CSR over j*N + k.")
    for n, ptr, ei, ec in tables:
        L.append(f"__device__ const int shv_mtab_ptr_{n}[{len(ptr)}] = {{" + ",".join(map(str, ptr)) + "};")
        L.append(f"__device__ const unsigned char shv_mtab_idx_{n}[{max(len(ei), 1)}] = {{" + ",".join(map(str, ei or [0])) + "};")
        L.append(f"__device__ const float shv_mtab_val_{n}[{max(len(ec), 1)}] = {{" + ",".join(flit(c) for c in (ec or [0.0])) + "};")
    L.append("")
    L.append("// Lighting-gradient contraction Lbar_i = sum_{j, kk} C_{i j k(kk)} Q[j][kk],")
    L.append("// Q over the transfer support (kk indexes the support); entries j * 32 + kk, row i's")
    L.append("// entries split over 4 threads (entry e of the row to thread e mod 4), padded per thread.")
    for n in range(1, MAX_BANDS + 1):
        N = n * n
        C = real_gaunt(n)
        supp = transfer_support(n)
        pos = {k: kk for kk, k in enumerate(supp)}
        rows = [[] for _ in range(N)]
        for (i, j, k), c in C.items():
            if k in pos:
                rows[i].append((j * 32 + pos[k], c))
        ptr, ent, val = [0], [], []
        for r in rows:
            for e, c in sorted(r):
                ent.append(e)
                val.append(c)
            ptr.append(len(ent))
        # Padded per-thread layout: thread (i, part) of the contraction takes
        # the entries ptr[i] + part, + 4, ... in order, as slots 0, 1, ...;
        # every (i, part) gets the same slot count (unused slots: entry 0,
        # value 0, beyond the count) so its loads can all be issued at once.
        slots = max([(ptr[i + 1] - ptr[i] - part + 3) // 4 for i in range(N) for part in range(4)] + [1])
        pent, pval, pcnt = [], [], []
        for i in range(N):
            for part in range(4):
                es = list(range(ptr[i] + part, ptr[i + 1], 4))
                pcnt.append(len(es))
                pent += [ent[e] for e in es] + [0] * (slots - len(es))
                pval += [val[e] for e in es] + [0.0] * (slots - len(es))
        L.append(f"static constexpr int SHV_LTAB_SLOTS_{n} = {slots};")
        L.append(f"__device__ const int shv_ltab_cnt_{n}[{len(pcnt)}] = {{" + ",".join(map(str, pcnt)) + "};")
        L.append(f"__device__ const unsigned short shv_ltab_pent_{n}[{len(pent)}] = {{" + ",".join(map(str, pent)) + "};")
        L.append(f"__device__ const float shv_ltab_pval_{n}[{len(pval)}] = {{" + ",".join(flit(c) for c in pval) + "};")
    L.append("")
    emit_quad(L)
    L.append("")
    emit_lat(L)
    emit_turns(L)
    L.append("")
    for n in range(1, MAX_BANDS + 1):
        supp = transfer_support(n)
        L.append(f"static constexpr int SHV_HSUPP_COUNT_{n} = {len(supp)};")
        L.append(f"static constexpr int SHV_HSUPP_{n}[{len(supp)}] = {{" + ",".join(map(str, supp)) + "};")
    open(path, "w").write("\n".join(L) + "\n")


def main():
    out = sys.argv[1] if len(sys.argv) > 1 else os.path.join(os.path.dirname(os.path.abspath(__file__)), "generated")
    os.makedirs(out, exist_ok=True)
    # self-checks of the derivation (selection rules and DC row)
    for n, nnz in ((4, 353), (6, 2907), (8, 12868)):
        C = real_gaunt(n)
        assert len(C) == nnz, (n, len(C))
        for j in range(n * n):
            assert abs(C.get((0, j, j), 0.0) - 1 / math.sqrt(4 * PI)) < 1e-14
    emit_constants(os.path.join(out, "shv_constants.h"))
    emit_gaunt(os.path.join(out, "shv_gaunt.h"))


if __name__ == "__main__":
    main()
