"""The host side of shade_sh and shade_sh_channels over the forms that inputs
come in: strides, types, empty sizes, edits after the forward pass, another
stream.  The values are FP32 numbers throughout, so every form has the bits of
plain FP32 rows; those are held against the C entry points."""
import numpy as np
import pytest
import torch

import scenegen
from gpu_helpers import run_render

pytestmark = pytest.mark.gpu

NAMES = ("points", "normals", "albedo", "spheres", "light")
P, S, N_BANDS, C = 333, 9, 4, 3


def _forms(x):
    wide = torch.zeros(2 * x.shape[0], *x.shape[1:], device=x.device)
    wide[::2] = x
    return {
        "rows": x,
        "columns": x.t().contiguous().t() if x.dim() == 2 else x,
        "every second": wide[::2],
        "float64": x.double(),
        "negated view": torch._neg_view(-x),
    }


def _inputs(channels):
    sc = scenegen.scene_random_shell(77, P, S, N_BANDS)
    t = {k: torch.tensor(np.asarray(sc[k], np.float32), device="cuda") for k in NAMES}
    t["points"] = t["points"].half().float()  # exact in every type below
    if channels:
        t["albedo"] = torch.stack([t["albedo"] * s for s in (1.0, 0.5, 0.25)], 1)
        t["light"] = torch.stack([t["light"] * s for s in (1.0, 2.0, 0.5)])
    g = torch.tensor(np.asarray(sc["grad_radiance"], np.float32), device="cuda")
    return t, (torch.stack([g, 2 * g, -g], 1) if channels else g)


def _run(op, t, g, between=None):
    xs = [t[k].detach().requires_grad_() for k in NAMES]
    y = op(*xs, N_BANDS)
    if between:
        between(xs)
    return [y.detach(), *torch.autograd.grad(y, xs, g.to(y.dtype))]


def _op(channels):
    from paper_2104_00359_amd import ops
    return ops.shade_sh_channels if channels else ops.shade_sh


@pytest.mark.parametrize("channels", [False, True])
@pytest.mark.parametrize("form", ["columns", "every second", "float64", "negated view"])
def test_forms_have_the_bits_of_plain_rows(form, channels):
    t, g = _inputs(channels)
    want = _run(_op(channels), t, g)
    # positions and normals in the form, each alone and both
    for which in (("points",), ("normals",), ("points", "normals")):
        got = _run(_op(channels), dict(t, **{k: _forms(t[k])[form] for k in which}), g)
        for a, b, k in zip(got, want, ("radiance",) + NAMES):
            assert torch.equal(a.float(), b), (which, k)


def test_plain_rows_have_the_bits_of_the_entry_points():
    t, g = _inputs(False)
    got = _run(_op(False), t, g)
    sc = dict({k: v.cpu().numpy() for k, v in t.items()}, n_bands=N_BANDS)
    ref = run_render(sc, g.cpu().numpy())
    for a, k in zip(got, ("B", "grad_points", "grad_normals", "grad_albedo", "grad_spheres", "grad_light")):
        assert np.array_equal(a.cpu().numpy(), ref[k]), k


@pytest.mark.parametrize("channels", [False, True])
def test_positions_may_change_after_the_forward_pass(channels):
    t, g = _inputs(channels)
    want = _run(_op(channels), t, g)
    t = {k: v.clone() for k, v in t.items()}

    def edit(xs):
        with torch.no_grad():
            xs[0].data.add_(1.0)
            xs[1].data.mul_(2.0)
    for a, b in zip(_run(_op(channels), t, g, edit), want):
        assert torch.equal(a, b)


@pytest.mark.parametrize("channels", [False, True])
def test_another_stream(channels):
    t, g = _inputs(channels)
    want = _run(_op(channels), t, g)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        got = _run(_op(channels), t, g)
    s.synchronize()
    for a, b in zip(got, want):
        assert torch.equal(a, b)


@pytest.mark.parametrize("p,s", [(0, S), (P, 0), (1, 1)])
def test_smallest_sizes(p, s):
    t, g = _inputs(False)
    t = dict(t, points=t["points"][:p], normals=t["normals"][:p], albedo=t["albedo"][:p], spheres=t["spheres"][:s])
    got = _run(_op(False), t, g[:p])
    assert [tuple(x.shape) for x in got] == [(p,), (p, 3), (p, 3), (p,), (s, 4), (N_BANDS ** 2,)]
    assert all(torch.isfinite(x).all() for x in got)


def test_refused_inputs_are_named():
    t, _ = _inputs(False)
    op = _op(False)
    with pytest.raises(ValueError, match="normals"):
        op(t["points"], t["normals"][:-1], t["albedo"], t["spheres"], t["light"], N_BANDS)
    with pytest.raises(ValueError, match="light"):
        op(*[t[k] for k in NAMES[:4]], t["light"][None], N_BANDS)
    with pytest.raises(RuntimeError, match="spheres"):
        op(t["points"], t["normals"], t["albedo"], t["spheres"].cpu(), t["light"], N_BANDS)
    with pytest.raises(RuntimeError, match=r"sh_render_forward: unsupported parameters \(-2\): n_squarings"):
        op(*[t[k] for k in NAMES], N_BANDS, -1.0, 99)
