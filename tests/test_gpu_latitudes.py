"""Products through latitudes (6 to 8 bands) at the edges of the receiver
tiles, in every kernel that uses them, against the FP64 oracle.

Tolerances as for the other exponential tests: V ||dV|| / ||V|| <= 1e-5,
gradients ||d grad|| / ||grad|| <= 1e-4 per parameter group."""
import numpy as np
import pytest

import scenegen
from gpu_helpers import collect, lib, rel_l2, run_hip, run_render
from oracle import method

pytestmark = pytest.mark.gpu

GRADS = ("grad_points", "grad_normals", "grad_albedo", "grad_spheres", "grad_light")


def _check(h, sc, mode="squaring"):
    o = method.run_forward_backward(sc, sc["grad_radiance"], exp_mode=mode)
    ev = rel_l2(h["V"], o["V"].numpy())
    assert ev <= 1e-5, ev
    for key in GRADS:
        e = rel_l2(h[key], o[key].numpy())
        assert e <= 1e-4, (key, e)


@pytest.mark.parametrize("n", [6, 7, 8])
@pytest.mark.parametrize("P", [1, 64, 65, 257])
def test_tile_edges_in_both_layouts(n, P):
    L = lib()
    sc = scenegen.scene_random_shell(600 + n, P, 21, n)
    four = run_render(sc, sc["grad_radiance"], flags=L.SHV_FLAG_EXP_FOUR_WAVES)
    _check(four, sc)
    one = run_render(sc, sc["grad_radiance"], flags=L.SHV_FLAG_EXP_ONE_WAVE)
    for key in ("V", "B") + GRADS:
        assert np.array_equal(one[key], four[key]), key


@pytest.mark.parametrize("n", [6, 7, 8])
@pytest.mark.parametrize("mode", ["taylor2", "product"])
def test_other_modes_at_a_ragged_tile(n, mode):
    L = lib()
    flags = L.SHV_FLAG_EXP_PRODUCT if mode == "product" else L.SHV_FLAG_EXP_TAYLOR | L.SHV_FLAG_EXP_TAYLOR_ORDER(2)
    sc = scenegen.scene_random_shell(700 + n, 65, 21, n)
    _check(run_hip(sc, sc["grad_radiance"], flags=flags), sc, mode)


def test_no_squarings_keep_the_linear_approximation():
    sc = scenegen.scene_random_shell(808, 65, 5, 8)
    sc["spheres"][:, 3] *= 0.2        # a small exponent, where k = 0 means something
    h = run_render(sc, sc["grad_radiance"], k=0)
    o = method.run_forward_backward(sc, sc["grad_radiance"], n_squarings=0)
    assert rel_l2(h["V"], o["V"].numpy()) <= 1e-5
    for key in GRADS:
        assert rel_l2(h[key], o[key].numpy()) <= 1e-4, key


@pytest.mark.parametrize("n,P", [(1, 1), (2, 65), (3, 64), (5, 63), (6, 129), (7, 65), (8, 1), (8, 129)])
def test_separable_quadrature_at_tile_edges(n, P):
    """Every number of waves per block and of latitudes per wave."""
    L = lib()
    sc = scenegen.scene_random_shell(900 + n, P, 13, n)
    _check(run_hip(sc, sc["grad_radiance"], flags=L.SHV_FLAG_EXP_QUADRATURE), sc, "quadrature")


@pytest.mark.parametrize("n", [7, 8])
def test_large_launches_keep_the_four_wave_bits(n):
    """From 98,304 receivers of a scene, or of a batch's four-wave group, a lane
    takes a whole receiver; below, and for a scene that asks for four waves, it
    does not.  Ragged ends, a range that starts inside its scene, and a small
    scene beside large ones, against the four-wave layout bit for bit."""
    import torch
    from paper_2104_00359_amd import batch, ops
    L = lib()
    dev = torch.device("cuda", 0)
    ops.ensure_init(dev)
    scenes = [scenegen.scene_random_shell(1000 + n + i, P, 3, n) for i, P in enumerate((98305, 33001, 65, 700))]
    flags = (0, 0, 0, L.SHV_FLAG_EXP_FOUR_WAVES)
    refs = [run_render(sc, sc["grad_radiance"], flags=L.SHV_FLAG_EXP_FOUR_WAVES) for sc in scenes]
    single = run_render(scenes[0], scenes[0]["grad_radiance"])
    bufs = [batch.scene_buffers(sc, dev, flags=f) for sc, f in zip(scenes, flags)]
    for b in bufs:
        b.allocate(dev)
    calls = [[bufs[0].record(0, 512, defer=True)],                                           # below the line
             [bufs[0].record(512, 98305), bufs[2].record(), bufs[3].record(), bufs[1].record()]]
    for recs in calls:
        tab = batch.Table(recs, dev)
        tab.forward(torch.cuda.current_stream())
        tab.backward(torch.cuda.current_stream())
    torch.cuda.synchronize()
    for got, ref in [(single, refs[0])] + [(collect(b), r) for b, r in zip(bufs, refs)]:
        for key in ("V", "B") + GRADS:
            assert np.array_equal(got[key], ref[key]), key


@pytest.mark.parametrize("n", [6, 7, 8])
@pytest.mark.parametrize("k", [0, 1, 2, 3])
def test_four_waves_at_every_parity_of_the_squarings(n, k):
    """The waves' exchange before, between and after k squarings."""
    L = lib()
    sc = scenegen.scene_random_shell(1100 + n, 65, 7, n)
    sc["spheres"][:, 3] *= 0.5
    four = run_render(sc, sc["grad_radiance"], k=k, flags=L.SHV_FLAG_EXP_FOUR_WAVES)
    one = run_render(sc, sc["grad_radiance"], k=k, flags=L.SHV_FLAG_EXP_ONE_WAVE)
    for key in ("V", "B") + GRADS:
        assert np.array_equal(one[key], four[key]), key
    assert all(np.isfinite(four[key]).all() for key in ("V", "B") + GRADS)
