"""Constants of the products through latitudes (csrc/gen_tables.py): the
transform, the Fourier product and the transposed transform built from them
are the Gaunt contraction, in 64 bits."""
import importlib.util
import math
import os

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2104_00359_amd", "csrc")


@pytest.fixture(scope="module")
def gen():
    spec = importlib.util.spec_from_file_location("gen_tables", os.path.join(CSRC, "gen_tables.py"))
    m = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(m)
    return m


def _fourier(e, row, n, sign):
    """c_m = A_m - i B_m, m = -(n-1) .. n-1, at +-z."""
    c = np.zeros(2 * n - 1, complex)
    for m in range(n):
        at = m * n - m * (m - 1) // 2
        q = [row[at + l - m] * (sign if (l - m) % 2 else 1.0) for l in range(m, n)]
        a = sum(t * e[l * l + l + m] for t, l in zip(q, range(m, n)))
        b = sum(t * e[l * l + l - m] for t, l in zip(q, range(m, n))) if m else 0.0
        c[n - 1 + m], c[n - 1 - m] = a - 1j * b, a + 1j * b
    return c


@pytest.mark.parametrize("n", [6, 7, 8])
def test_product_through_latitudes_is_the_gaunt_contraction(gen, n):
    N = n * n
    rng = np.random.default_rng(n)
    a, b = rng.standard_normal((2, N))
    want = np.zeros(N)
    for (i, j, k), v in gen.real_gaunt(n).items():
        want[i] += v * a[j] * b[k]
    scale = np.array([(1.0 if gen.lm(i)[1] == 0 else math.sqrt(0.5)) / math.sqrt(4 * math.pi) for i in range(N)])
    pairs, eq = gen.lat_rows(n)
    got = np.zeros(N)
    for row, signs in [(r, (1, -1)) for r in pairs] + [(r, (1,)) for r in eq]:
        for s in signs:
            d = np.convolve(_fourier(a * scale, row, n, s), _fourier(b * scale, row, n, s))[n - 1:-(n - 1)]
            for m in range(n):
                at = m * n - m * (m - 1) // 2
                for l in range(m, n):
                    t = row[at + l - m] * (s if (l - m) % 2 else 1.0)
                    got[l * l + l + m] += t * d[n - 1 + m].real
                    if m:
                        got[l * l + l - m] += -t * d[n - 1 + m].imag
    # the weight holds a factor 2: twice the product; 1e-13 is a few hundred roundings of 1e-16
    assert np.allclose(got / scale, 2 * want, rtol=0, atol=1e-13 * np.abs(want).max() * N)


@pytest.mark.parametrize("n", [6, 7, 8])
def test_output_groups_are_whole_orders(gen, n):
    for groups in (gen.forward_groups(n), gen.adjoint_groups(n)):
        assert sorted(i for g in groups for i in g) == list(range(n * n))
        owner = {abs(gen.lm(i)[1]): g for g, members in enumerate(groups) for i in members}
        assert all(owner[abs(gen.lm(i)[1])] == g for g, members in enumerate(groups) for i in members)


def test_sphere_frame_rotation_and_its_generators(gen):
    """R = K^-1 Z(-theta) K Z(-phi) takes the direction (theta, phi) to +z, and the generators used by the
    adjoint are the derivatives of the rotations about x and y; 1e-12 is a few thousand roundings of 64 bits."""
    n = gen.MAX_BANDS
    K = gen.quarter_turn()
    assert np.allclose(K @ K.T, np.eye(n * n), atol=1e-12)
    assert all(K[i, j] == 0 for i in range(n * n) for j in range(n * n) if gen.lm(i)[0] != gen.lm(j)[0])
    for th, ph in ((0.7, 1.9), (0.0, 0.0), (math.pi, -2.0), (1.3, 0.4)):
        d = np.array([math.sin(th) * math.cos(ph), math.sin(th) * math.sin(ph), math.cos(th)])
        f = K.T @ gen.z_turn(-th) @ K @ gen.z_turn(-ph) @ gen.real_basis(d, n)
        want = [math.sqrt((2 * gen.lm(i)[0] + 1) / (4 * math.pi)) if gen.lm(i)[1] == 0 else 0.0 for i in range(n * n)]
        assert np.allclose(f, want, atol=1e-12)
    Lz = gen.z_turn(0.0, True)
    A = K.T @ gen.z_turn(-math.pi / 2) @ K
    rng = np.random.default_rng(1)
    f, d = rng.standard_normal(n * n), rng.standard_normal((7, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    # (L f)(w) = -(axis x w) . grad f; the coordinates' own functions (band 1) give it exactly
    for L, axis in ((A.T @ Lz @ A, (1.0, 0, 0)), (K.T @ Lz @ K, (0, 1.0, 0)), (Lz, (0, 0, 1.0))):
        for c in range(3):
            e = np.zeros(n * n)
            e[(3, 1, 2)[c]] = math.sqrt(4 * math.pi / 3)   # the function w -> w_c
            assert np.allclose(gen.real_basis(d, n) @ (L @ e), -np.cross(axis, d)[:, c], atol=1e-12)


@pytest.mark.parametrize("n", [6, 7, 8])
def test_waves_of_the_product_chain_own_every_band_and_order(gen, n):
    bands, orders = gen.turn_groups(n)
    assert len(bands) == len(orders) == n and set(bands) == set(orders) == {0, 1, 2, 3}
