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
