"""Algorithmic work per unit for each kernel (used for roofline figures).

Counting rule: one floating-point add, multiply, square root, reciprocal
square root or exponential = 1 flop; a fused multiply-add = 2 flops.  The
counts are those of the minimal operation graph of the formulation the
kernels implement (polynomial SH basis, sparse triple products up to 5 bands,
products through latitudes above); lane-level
overheads (index arithmetic, cross-lane reductions, tail lanes) are not
counted.  Units: one (receiver, sphere) pair for the pair kernels, one
receiver for the per-receiver kernels.
"""
from __future__ import annotations

import functools
import os
import sys


def _tri(n):
    return n * (n - 1) // 2


def _basis_flops(n: int) -> int:
    """One pair's basis: the cap's terms a_l(t), Re / Im (x + i y)^m, p_l(z)
    and the rows rho_l^m of the orders 1 .. n - 1."""
    cap = (1 if n > 2 else 0) + 3 * max(n - 3, 0)
    cs = 6 * max(n - 2, 0)
    p = (2 if n > 2 else 0) + 3 * max(n - 3, 0)
    rows = 2 * _tri(max(n - 2, 0))              # one FMA per l >= m + 2
    return cap + cs + p + rows


def pair_fwd_flops(n: int) -> int:
    geom = 21                                   # c - x, |v|^2, rsqrt, s, r/d, its square, 1 - s^2, sqrt, u
    u = _tri(max(n - 1, 0))                     # a_l rho_l^m for l > m >= 1
    acc = 4 + 2 * (n - 1) + 4 * _tri(n)         # compensated DC, m = 0, m > 0 two FMAs each
    return geom + _basis_flops(n) + u + acc


def pair_bwd_flops(n: int) -> int:
    geom = 18
    m0 = 2 * max(n - 1, 0)                      # f_l and h_l of order 0
    lm = 0
    for m in range(1, n):
        for l in range(m, n):
            lm += 3 + 4                         # b, X
            lm += 1 if l == m else 2 + 1        # f; v
            lm += 0 if l == m else 1 if l == m + 1 else 2 + (1 if (l - m) % 2 == 0 else 0)  # h
    comb = 10 * max(n - 2, 0)                   # per-order combination into Gx, Gy
    ends = (2 if n > 2 else 0) + 3 * max(n - 3, 0) + 5 * max(n - 1, 0) + 1  # p_l(t), Gz, Gt
    chain = 26 + 3 + 4                          # tangent projection, t chain, receiver / sphere sums
    return geom + _basis_flops(n) + m0 + lm + comb + ends + chain


# Products through latitudes (6 bands and above): per row +-z or z = 0, the
# transforms up of the factors, the Fourier product, the transform down.
LAT_MIN_BANDS = 6


def _lat_up_flops(n: int, eq: bool, mean: bool) -> int:
    f = 0
    for m in range(n):
        terms = [0, 0]
        for l in range(m, n):
            odd = (l - m) % 2
            if (l == 0 and not mean) or (eq and odd):
                continue
            terms[odd] += 1
        parts = 1 if m == 0 else 2              # cosine (and sine)
        f += parts * sum(2 * t - 1 for t in terms if t)
        f += 0 if eq else 2 * parts             # the sum and the difference
    return f


def _lat_conv_flops(n: int, square: bool) -> int:
    f = 0
    for m in range(n):
        if square:
            if m == 0:
                f += 2 + 4 * (n - 1)
                continue
            f += 2
            for t in range(1, m // 2 + 1):
                f += 8 if 2 * t < m else 8
            f += 8 * (n - 1 - m)
        else:
            if m == 0:
                f += 3 + 4 * (n - 1)
                continue
            f += 6 + 8 * (m - 1) + 16 * (n - 1 - m)
    return f


def _lat_down_flops(n: int, eq: bool) -> int:
    f = 0
    for m in range(n):
        parts = 1 if m == 0 else 2
        f += parts * (0 if eq else 2)
        f += 2 * parts * sum(1 for l in range(m, n) if not (eq and (l - m) % 2))
    return f


@functools.lru_cache(maxsize=None)
def _lat_flops(n: int, square: bool) -> int:
    pairs, eq = (len(r) for r in _tables().lat_rows(n))
    f = 2 * n * n
    for count, at_eq in ((pairs, False), (eq, True)):
        row = _lat_up_flops(n, at_eq, False) + (0 if square else _lat_up_flops(n, at_eq, True))
        row += (1 if at_eq else 2) * _lat_conv_flops(n, square) + _lat_down_flops(n, at_eq)
        f += count * row
    return f


def _tables():
    here = os.path.join(os.path.dirname(os.path.abspath(__file__)), "csrc")
    if here not in sys.path:
        sys.path.insert(0, here)
    import gen_tables  # the library's own table generator
    return gen_tables


@functools.lru_cache(maxsize=None)
def _gaunt_counts(n: int):
    gen_tables = _tables()
    C = gen_tables.real_gaunt(n)
    sym = [(i, j, k) for (i, j, k) in C if j <= k]
    pairs = {(j, k) for (_, j, k) in sym}
    upairs = {(i, k) for (_, i, k) in C if i <= k}
    supp = set(gen_tables.transfer_support(n))
    vh = [(i, j, k) for (i, j, k) in C if k in supp]
    vh_pairs = {(j, k) for (_, j, k) in vh}
    return dict(nnz=len(C), sym=len(sym), pairs=len(pairs), upairs=len(upairs),
                diag=sum(1 for (i, k) in upairs if i == k), vh=len(vh), vh_pairs=len(vh_pairs),
                supp=len(supp))


def square_flops(n: int) -> int:
    if n >= LAT_MIN_BANDS:
        return _lat_flops(n, True)
    c = _gaunt_counts(n)
    return c["pairs"] + 2 * c["sym"]


def square_adj_flops(n: int) -> int:
    if n >= LAT_MIN_BANDS:
        return _lat_flops(n, False)
    c = _gaunt_counts(n)
    off = c["upairs"] - c["diag"]
    return c["diag"] + 3 * off + 2 * c["sym"]


def exp_fwd_flops(n: int, k: int) -> int:
    N = n * n
    prologue = 3 * N + 2 * N + 4                # scale, |G|^2, exp, a * G
    return prologue + k * square_flops(n) + N + 1


def exp_bwd_flops(n: int, k: int) -> int:
    N = n * n
    return 3 * N + 2 + k * square_adj_flops(n) + 2 * N + 5 * N


def shade_fwd_flops(n: int) -> int:
    c = _gaunt_counts(n)
    N = n * n
    return 12 + 3 * N + c["supp"] * (2 * N + 2) + 1


def shade_bwd_flops(n: int) -> int:
    c = _gaunt_counts(n)
    N = n * n
    h = 12 + 3 * N
    mv = c["supp"] * (2 * N + 3)
    vbar = N * (2 * c["supp"] + 1)
    nbar = 10 * N + 15
    lbar = c["supp"] + 2 * N * c["supp"]        # w H, then the Q GEMM (contraction with C is per call)
    return h + mv + vbar + nbar + lbar


def shade_ch_fwd_flops(n: int, channels: int) -> int:
    """Several channels: the transfer once, V^T M_c H per channel."""
    c = _gaunt_counts(n)
    N = n * n
    return 12 + 3 * N + channels * (c["supp"] * (2 * N + 2) + 1)


def shade_ch_bwd_flops(n: int, channels: int) -> int:
    """Several channels: the transfer and the normal cotangent once, the
    shading value, V and H cotangents and the lighting GEMM per channel (the
    channel sums of the V and H cotangents are one add per entry)."""
    c = _gaunt_counts(n)
    N = n * n
    h = 12 + 3 * N
    mv = c["supp"] * (2 * N + 4)
    vbar = N * (2 * c["supp"] + 2)
    nbar = 10 * N + 15
    lbar = c["supp"] + 2 * N * c["supp"]
    return h + nbar + channels * (mv + vbar + lbar)


def _quad_flops(n: int, evaluations: int, per_node: int) -> int:
    """Per receiver, the separable 4n x 8n rule: at each latitude
    ``evaluations`` Fourier sums up and to the azimuths (folded into a quarter,
    8 additions per four azimuths), ``per_node`` flops at a node, and one sum
    back."""
    transform = _lat_up_flops(n, False, True)   # of a pair of latitudes
    down = _lat_down_flops(n, False)
    azimuths = 2 * n * (2 * (2 * n - 1) + 8)
    return 2 * n * (evaluations * transform + down) + 4 * n * ((evaluations + 1) * azimuths + 8 * n * per_node)


def exp_quad_fwd_flops(n: int) -> int:
    """f at the nodes, one exponential (and the weight of the latitude, once
    per Fourier sum) and V."""
    return _quad_flops(n, 1, 1)


def exp_quad_bwd_flops(n: int) -> int:
    """f and g = Vbar at the nodes, exp(f) g, and Fbar."""
    return _quad_flops(n, 2, 2)


def exp_taylor_fwd_flops(n: int, k: int, K: int) -> int:
    """Per receiver: the DC split and scaling (2 N), K Horner steps (one
    sparse product each, returned doubled, and its scale), k squarings and
    the final exp(c) scale."""
    N = n * n
    return 2 * N + K * (square_adj_flops(n) + N) + k * square_flops(n) + N + 1


def exp_taylor_bwd_flops(n: int, k: int, K: int) -> int:
    """Per receiver: cbar and exp(c) Vbar (3 N), k adjoint squarings, the
    Horner adjoint (two sparse products per step but one in the last, each
    with its scale / accumulation) and the weights W (2 N)."""
    N = n * n
    return 3 * N + k * square_adj_flops(n) + (2 * K - 1) * (square_adj_flops(n) + 2 * N) + 2 * N


@functools.lru_cache(maxsize=None)
def _turn_flops(n: int) -> int:
    """One rotation of a vector into a sphere's frame (or back): two turns
    about z and two quarter turns."""
    quarter = 2 * int((abs(_tables().quarter_turn()[:n * n, :n * n]) > 1e-12).sum()) - n * n
    return 2 * (6 * _tri(n) + quarter)


def _zonal_flops(n: int) -> int:
    """A product with a zonal function in its frame: the rows up, a multiply
    per Fourier coefficient and sign, and down."""
    pairs, eq = (len(r) for r in _tables().lat_rows(n))
    return (pairs * (_lat_up_flops(n, False, True) + 2 * (2 * n - 1) + _lat_down_flops(n, False) + 4 * n)
            + eq * (_lat_up_flops(n, True, True) + 2 * n - 1 + _lat_down_flops(n, True) + n))


def prod_fwd_flops(n: int) -> int:
    """Per (receiver, sphere) step of the direct product chain: from 6 bands
    up the vector turned into the sphere's frame, multiplied by the zonal
    blocker and turned back; below, the pair's blocker vector, one sparse
    product V * h and the update."""
    N = n * n
    if n >= LAT_MIN_BANDS:
        return 60 + 2 * _turn_flops(n) + _zonal_flops(n) + 2 * N
    return pair_fwd_flops(n) + N + square_adj_flops(n) + 2 * N


def prod_bwd_flops(n: int) -> int:
    """Per step of the chain's adjoint: from 6 bands up the state and its
    cotangent turned, the zonal product's adjoint, the tangential derivatives
    and the turn back; below, the blocker vector again, two sparse products,
    the pair weights and the pair adjoint."""
    N = n * n
    if n >= LAT_MIN_BANDS:
        return 100 + 3 * _turn_flops(n) + 2 * _zonal_flops(n) + 8 * N
    return (pair_fwd_flops(n) + N) + 2 * square_adj_flops(n) + 3 * N + 2 * N + pair_bwd_flops(n)


def envmap_pixel_flops(n: int) -> int:
    """One map pixel: 2n - 1 FMAs, and a fourth (rows of a block share it) of
    its column's sine and cosine and their 2n - 4 multiples."""
    return 2 * (2 * n - 1) + (4 + 6 * max(n - 2, 0)) // 4


# Bytes each kernel must move to / from HBM per unit (FP32).
def exp_fwd_bytes(n: int, k: int, nchunks: int) -> int:
    N = n * n
    return 4 * (nchunks * N + N + 1 + k * N)


def pair_fwd_bytes_per_receiver(n: int, nchunks: int) -> int:
    return 4 * (3 * nchunks + n * n * nchunks)


def exp_shade_bwd_bytes(n: int, k: int) -> int:
    """Algorithmic HBM bytes per receiver of the fused exponential + shading
    adjoint: it reads the radiance cotangent, V, the saved c and E_0 ..
    E_{k-1}, the normal and the albedo, and writes W (the cotangent of F'),
    the normal and albedo gradients and its share of the per-tile lighting
    partials (N floats per 64 receivers)."""
    N = n * n
    reads = 4 * (1 + N + (1 + k * N) + 3 + 1)
    writes = 4 * (N + 3 + 1) + 4 * N / 64
    return int(round(reads + writes))


def kernel_work(name: str, n: int, k: int, P: int, S: int, channels: int = 1, pixels: int = 0, order: int = 0):
    """(flops, unit count) of one launch of kernel ``name`` (``channels``
    for the multi-channel shading kernels, ``pixels`` = C H W for the
    environment-map projection, ``order`` = K of the Taylor exponential)."""
    if name == "exp_taylor_fwd":
        return exp_taylor_fwd_flops(n, k, order) * P, P
    if name == "exp_taylor_bwd":
        return exp_taylor_bwd_flops(n, k, order) * P, P
    if name == "shade_ch_fwd":
        return shade_ch_fwd_flops(n, channels) * P, P
    if name == "shade_ch_bwd":
        return shade_ch_bwd_flops(n, channels) * P, P
    if name == "envmap_rows":
        return envmap_pixel_flops(n) * pixels, pixels
    if name == "exp_quad_fwd":
        return exp_quad_fwd_flops(n) * P, P
    if name == "exp_quad_bwd":
        return exp_quad_bwd_flops(n) * P, P
    if name in ("prod_fwd", "prod_fwd_states"):
        return prod_fwd_flops(n) * P * S, P * S
    if name == "prod_bwd":
        return prod_bwd_flops(n) * P * S, P * S
    if name == "pair_fwd":
        return pair_fwd_flops(n) * P * S, P * S
    if name == "pair_bwd":
        return pair_bwd_flops(n) * P * S, P * S
    if name == "exp_fwd":
        return exp_fwd_flops(n, k) * P, P
    if name == "exp_bwd":
        return exp_bwd_flops(n, k) * P, P
    if name == "shade_fwd":
        return shade_fwd_flops(n) * P, P
    if name == "shade_bwd":
        return shade_bwd_flops(n) * P, P
    if name == "exp_shade_fwd":
        return (exp_fwd_flops(n, k) + shade_fwd_flops(n)) * P, P
    if name == "exp_shade_bwd":
        return (exp_bwd_flops(n, k) + shade_bwd_flops(n)) * P, P
    return None, None


BATCH_KERNELS = {"batch_pair_fwd": "pair_fwd", "batch_pair_bwd": "pair_bwd", "batch_exp_shade_fwd": "exp_shade_fwd",
                 "batch_exp_shade_bwd": "exp_shade_bwd"}


def batch_work(name: str, scenes):
    """(flops, unit count) of all launches of batched kernel ``name`` in one
    batched call over ``scenes`` (tuples (n, k, P, S)).  A name carrying a
    band count ("batch_pair_bwd/n8", "batch_exp_shade_fwd/n4/one") counts the
    scenes with that many bands only."""
    parts = name.split("/")
    single = BATCH_KERNELS.get(parts[0])
    if single is None:
        return None, None
    only = int(parts[1][1:]) if len(parts) > 1 and parts[1].startswith("n") else None
    flops = units = 0
    for n, k, P, S in scenes:
        if only is not None and n != only:
            continue
        f, u = kernel_work(single, n, k, P, S)
        flops += f
        units += u
    return flops, units
