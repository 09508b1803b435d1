"""The pair kernels' recurrences and constants against Legendre polynomials in
64 bits: zonal terms, rows, their derivatives, and the factor that turns their
product into g_l(t) y_lm."""
import math
import os
import sys

import numpy as np
import pytest
from numpy.polynomial import legendre, polynomial

sys.path.insert(0, os.path.join(os.path.dirname(__file__), "..", "paper_2104_00359_amd", "csrc"))
import gen_tables as gt  # noqa: E402

B = gt.MAX_BANDS
PAIR, ROW, ROW_K, ROW_0, CAP_B, LEG_B = gt.pair_constants()


def _q(l, m):
    """Coefficients of d^m P_l / dz^m."""
    c = legendre.leg2poly([0] * l + [1])
    return polynomial.polyder(c, m) if m else c


def _monic(l, z):
    r = [np.ones_like(z), z]
    for i in range(1, B - 1):
        r.append(z * r[i] - LEG_B[i] * r[i - 1])
    return r[l]


def _row(m, z):
    """rho_l^m for every l."""
    rows = [_monic(l, z) for l in range(B)]
    for k in range(1, m + 1):
        below, rows = rows, [None] * B
        for l in range(k, B):
            rows[l] = (np.ones_like(z) if l == k else z if l == k + 1
                       else rows[l - 2] + ROW[l][k] * below[l - 1])
    return rows


@pytest.mark.parametrize("l", range(B))
def test_pair_basis(l):
    z = np.linspace(-1, 1, 41)
    t = np.linspace(0, 1, 41)
    a = [1 - t, 1 - t * t, t * (1 - t * t)]
    for i in range(2, B - 1):
        a.append(t * a[i] - CAP_B[i] * a[i - 1])
    p = lambda k: polynomial.polyval(t, _q(k, 0)) if k >= 0 else np.ones_like(t)  # noqa: E731
    g = -2 * math.pi / (2 * l + 1) * (p(l - 1) - p(l + 1))
    lead = _q(l, 0)[-1]
    for m in range(l + 1):
        rho = _row(m, z)[l]
        norm = math.sqrt((2 * l + 1) / (4 * math.pi) * math.factorial(l - m) / math.factorial(l + m) * (2 if m else 1))
        want = np.outer(g, norm * polynomial.polyval(z, _q(l, m)))
        np.testing.assert_allclose(PAIR[l][m] * np.outer(a[l], rho), want, rtol=0, atol=1e-12 * np.abs(want).max())
        if l > m:  # d rho_l^m / dz in terms of rho_l^{m+1}
            c = ROW_0[l] if m == 0 else 1.0 if (l - m) % 2 else ROW_K[m]
            scale = 1 / lead if m == 0 else rho[-1] / polynomial.polyval(1.0, _q(l, m))
            d = scale * polynomial.polyval(z, _q(l, m + 1))
            np.testing.assert_allclose(c * _row(m + 1, z)[l], d, rtol=0, atol=1e-12 * np.abs(d).max())
    # d a_l / dt = -(l + 1) p_l(t)
    da = -np.ones_like(t) if l == 0 else polynomial.polyval(t, polynomial.polyder(
        polynomial.polymul([1, 0, -1], _q(l, 1) / _q(l, 1)[-1])))
    np.testing.assert_allclose(-(l + 1) * _monic(l, t), da, rtol=0, atol=1e-12 * np.abs(da).max())


def test_weights_are_exact_to_two_floats():
    """PAIR and its rest add up to the 64-bit factor (two 24-bit significands: 2^-48
    relative), and the DC factor over sqrt(4 pi) is exactly -1/2."""
    for l in range(B):
        for m in range(l + 1):
            hi, lo = np.float32(PAIR[l][m]), np.float32(gt.float32_rest(PAIR[l][m]))
            assert abs(float(hi) + float(lo) - PAIR[l][m]) <= 2.0 ** -48 * abs(PAIR[l][m])
    assert np.float32(PAIR[0][0] / math.sqrt(4 * math.pi)) == np.float32(-0.5)
