"""Workloads of the soft-shadow library, through its public entry points.

Each case is a call (or the fixed group of calls) that a program makes over and
over: rendering a scene and its gradients, a batch of scenes, colour channels,
the other ways of forming the visibility, an environment map, one iteration of
the inverse problem, the rasteriser.  ``prepare`` makes the inputs on the GPU
from a seed, ``run`` is one pass, ``work`` counts what a pass cannot do without
and ``exact`` gives the same outputs by plain torch in 64 bits.
"""
import math
import random

import numpy as np
import torch

from paper_2104_00359_amd import _lib, batch, inverse, ops

EPS = 3.0
SQRT_4PI = math.sqrt(4.0 * math.pi)
F64 = torch.float64


def listed():
    body = dict(scene="body", P=20000, S=128, n=8, k=4)
    return [
        # A few hundred receivers in an optimisation loop: launches and host work are all there is.
        dict(name="shade_small", kind="shade", scene="shell", P=300, S=16, n=4, k=4),
        # The ordinary training step: a body's surface under its own fitted spheres, gradients to every input.
        dict(name="shade_body", kind="shade", **body),
        # The same body from a program that keeps its buffers and calls the C entry points.
        dict(name="render_body", kind="render", **body),
        # An image-space G-buffer, one receiver per pixel, resident buffers through the C entry points.
        dict(name="render_gbuffer", kind="render", scene="plane", P=512 * 512, S=256, n=8, k=4),
        # Rendering only (no state kept), a ragged receiver count and sphere count, 6 bands.
        dict(name="forward_ragged", kind="forward", scene="shell", P=50021, S=97, n=6, k=4),
        # The serving and benchmark step: 64 independent scenes replayed from one graph.
        dict(name="batch64", kind="batch", scenes=64, P=50000, S=256, n=0, k=4),
        # RGB: three channels through one visibility, forward and backward.
        dict(name="rgb_body", kind="rgb", C=3, **body),
        # The accurate visibility modes, forward and backward.
        dict(name="quadrature_body", kind="mode", mode="quadrature", **body),
        dict(name="product_body", kind="mode", mode="product", **body),
        # A captured environment map onto the lighting.
        dict(name="envmap", kind="envmap", C=3, H=512, W=1024, n=8),
        # One gradient-descent iteration of the inverse problem: deform, render, loss, adjoints, update.
        dict(name="inverse_body", kind="inverse", K=625, **body),
        # The shaded mesh into a 512 x 512 image and back to its vertices.
        dict(name="raster_mesh", kind="raster", parts=24, rings=29, segments=30, size=512),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["shade", "shade", "shade", "render", "render", "forward", "batch", "rgb", "mode", "mode",
                       "envmap", "inverse", "raster"])
    n = rng.choice([2, 3, 4, 4, 5, 6, 6, 7, 8, 8, 8])
    k = rng.choice([3, 4, 4, 4, 4, 5])
    scene = rng.choice(["shell", "shell", "body", "plane"])
    if kind in ("shade", "render", "forward"):
        P = _log_int(rng, 65, 200000)
        S = _log_int(rng, 5, min(512, 60_000_000 // P))
        return dict(kind=kind, scene=scene, P=P, S=S, n=n, k=k)
    if kind == "batch":
        return dict(kind=kind, scenes=rng.randint(2, 48), P=_log_int(rng, 5200, 50000), S=rng.randint(40, 256), n=0,
                    k=k)
    if kind == "rgb":
        return dict(kind=kind, C=rng.randint(1, 4), scene=scene, P=_log_int(rng, 300, 100000),
                    S=_log_int(rng, 8, 256), n=n, k=k)
    if kind == "mode":
        mode = rng.choice(["quadrature", "product", "taylor1", "taylor2", "taylor3"])
        P = _log_int(rng, 200, 20000)
        return dict(kind=kind, mode=mode, scene=scene, P=P, S=_log_int(rng, 8, 128), n=n, k=k)
    if kind == "envmap":
        H = _log_int(rng, 16, 1024)
        return dict(kind=kind, C=rng.randint(1, 4), H=H, W=2 * H + rng.choice([0, 0, 1, 3]), n=n)
    if kind == "inverse":
        P, S = _log_int(rng, 300, 40000), _log_int(rng, 8, 128)
        return dict(kind=kind, scene="body", P=P, S=S, n=n, k=k, K=max(1, 4 * P // S))
    return dict(kind="raster", parts=rng.randint(4, 30), rings=rng.randint(8, 30), segments=rng.randint(8, 32),
                size=_log_int(rng, 60, 900))


# ------------------------------------------------------------------ inputs

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 13)


def _dirs(g, m):
    d = torch.randn(m, 3, generator=g, device="cuda", dtype=F64)
    return d / d.norm(dim=1, keepdim=True)


def _uniform(g, lo, hi, *shape):
    return lo + (hi - lo) * torch.rand(*shape, generator=g, device="cuda", dtype=F64)


#: A standing figure: bones (A, B, radius) in metres, the second half mirrored in x.
_BONES = [((0, 0, 1.60), (0, 0, 1.72), .10), ((0, 0, 1.47), (0, 0, 1.56), .05), ((-.12, 0, 1.36), (.12, 0, 1.36), .12),
          ((0, 0, 1.10), (0, 0, 1.32), .13), ((0, .04, 1.02), (0, .04, 1.12), .10), ((-.09, 0, .98), (.09, 0, .98), .11)]
_PAIRS = [((.03, 0, 1.45), (.18, 0, 1.44), .045), ((.20, 0, 1.42), (.24, 0, 1.16), .045),
          ((.24, 0, 1.14), (.26, .06, .90), .035), ((.26, .07, .87), (.27, .09, .78), .03),
          ((.07, -.06, .93), (.07, -.06, .85), .08), ((.09, 0, .93), (.10, .02, .53), .075),
          ((.10, .02, .50), (.10, 0, .10), .05), ((.10, -.03, .05), (.11, .15, .04), .035),
          ((.11, .16, .035), (.11, .22, .03), .025)]


def _bones():
    b = list(_BONES)
    for A, B, r in _PAIRS:
        b += [(A, B, r), ((-A[0], A[1], A[2]), (-B[0], B[1], B[2]), r)]
    t = torch.tensor([[*A, *B, r] for A, B, r in b], dtype=F64, device="cuda")
    return t[:, :3], t[:, 3:6], t[:, 6]


def _scene(case, seed):
    """points [P, 3], normals [P, 3], albedo [P], spheres [S, 4], light [N], cotangent [P] in float32."""
    g, P, S, n = _gen(seed), case["P"], case["S"], case["n"]
    if case["scene"] == "shell":      # receivers on a unit ball, occluders floating around it
        pts = _dirs(g, P)
        nrm = pts
        r = _uniform(g, 0.05, 0.3, S)
        rho = ((1.05 + r) ** 3 + _uniform(g, 0, 1, S) * (8.0 - (1.05 + r) ** 3)) ** (1 / 3)
        sph = torch.cat([_dirs(g, S) * rho[:, None], r[:, None]], 1)
    elif case["scene"] == "plane":    # top-down view of spheres resting on the ground
        r = _uniform(g, 0.05, 0.25, S)
        xy = _uniform(g, -1, 1, S, 2)
        sph = torch.cat([xy, r[:, None], r[:, None]], 1)
        rows = max(1, int(math.isqrt(P)))
        i = torch.arange(P, device="cuda")
        X = ((i % rows) + 0.5) / rows * 2 - 1
        Y = ((i // rows) + 0.5) / math.ceil(P / rows) * 2 - 1
        X, Y = X.double(), Y.double()
        z = torch.zeros(P, device="cuda", dtype=F64)
        nrm = torch.zeros(P, 3, device="cuda", dtype=F64)
        nrm[:, 2] = 1
        for c in sph:
            h2 = c[3] ** 2 - (X - c[0]) ** 2 - (Y - c[1]) ** 2
            top = c[2] + h2.clamp(min=0).sqrt()
            hit = (h2 >= 0) & (top > z)
            z = torch.where(hit, top, z)
            nrm = torch.where(hit[:, None], (torch.stack([X, Y, top], 1) - c[:3]) / c[3], nrm)
        pts = torch.stack([X, Y, z], 1) + 1e-3 * nrm
    else:                             # a body: receivers on capsules, spheres of 0.9 R filling them
        A, B, R = _bones()
        ln = (B - A).norm(dim=1)
        share = torch.cumsum((ln + 2 * R) / R, 0)
        at = (torch.arange(S, device="cuda", dtype=F64) + 0.5) / S * share[-1]
        j = torch.searchsorted(share, at).clamp(max=len(R) - 1)
        before = torch.where(j > 0, share[(j - 1).clamp(min=0)], torch.zeros_like(at))
        f = (at - before) / (share[j] - before)
        sph = torch.cat([A[j] + f[:, None] * (B - A)[j], 0.9 * R[j][:, None]], 1)
        sph[:, :3] += 0.02 * R[j][:, None] * torch.randn(S, 3, generator=g, device="cuda", dtype=F64)
        area = ln * R + 2 * R * R
        m = 4 * P + 256
        b = torch.multinomial(area, m, replacement=True, generator=g)
        d = _dirs(g, m)
        ax = (B - A)[b] / ln[b][:, None]
        side = d - (d * ax).sum(1, keepdim=True) * ax
        side = side / side.norm(dim=1, keepdim=True)
        tube = torch.rand(m, generator=g, device="cuda", dtype=F64) < (ln * R / area)[b]
        u = torch.rand(m, generator=g, device="cuda", dtype=F64)
        end = torch.where(((d * ax).sum(1) > 0)[:, None], B[b], A[b])
        nrm = torch.where(tube[:, None], side, d)
        pts = torch.where(tube[:, None], A[b] + u[:, None] * (B - A)[b], end) + R[b][:, None] * nrm
        rel = pts[:, None] - A[None]
        tt = ((rel * (B - A)[None]).sum(-1) / (ln * ln)).clamp(0, 1)
        free = (rel - tt[..., None] * (B - A)[None]).norm(dim=-1) >= R * (1 - 1e-9)
        keep = (free | (torch.arange(len(R), device="cuda")[None] == b[:, None])).all(1)
        first = torch.argsort(~keep, stable=True)[:P]      # receivers inside no other bone first
        pts, nrm = pts[first] + 1e-3 * nrm[first], nrm[first]
    L = torch.randn(n * n, generator=g, device="cuda", dtype=F64)
    L[0] = 3.0
    out = dict(points=pts, normals=nrm, albedo=_uniform(g, 0.2, 0.9, P), spheres=sph, light=L,
               cotangent=torch.randn(P, generator=g, device="cuda", dtype=F64))
    return {key: v.float().contiguous() for key, v in out.items()}


INPUTS = ("points", "normals", "albedo", "spheres", "light")


def _batch_cases(case):
    """The scenes of a batch: their sizes belong to the case, their contents to the seed."""
    r = random.Random(case["scenes"] * 1_000_003 + case["P"] * 101 + case["S"])
    return [dict(kind="render", scene="shell", P=r.randint(5000, case["P"]), S=r.randint(32, case["S"]),
                 n=r.choice([4, 6, 8]), k=case["k"]) for _ in range(case["scenes"])]


def _rgb(case, seed):
    s, g, C = _scene(case, seed), _gen(seed + 1), case["C"]
    light = torch.randn(C, case["n"] ** 2, generator=g, device="cuda")
    light[:, 0] = 3.0
    s.update(albedo=_uniform(g, 0.2, 0.9, case["P"], C).float(), light=light,
             cotangent=torch.randn(case["P"], C, generator=g, device="cuda"))
    return s


def _image(case, seed):
    g, C, H, W = _gen(seed), case["C"], case["H"], case["W"]
    th = (torch.arange(H, device="cuda") + 0.5)[:, None] * (math.pi / H)
    ph = (torch.arange(W, device="cuda") + 0.5)[None] * (2 * math.pi / W)
    d = torch.stack([th.sin() * ph.cos(), th.sin() * ph.sin(), th.cos() + 0 * ph], -1)
    img = 0.3 + 0.7 * d[..., 2].clamp(min=0)[None] * _uniform(g, 0.5, 1.0, C, 1, 1)
    img = img * (1 + 0.2 * torch.cos(2 * ph + _uniform(g, 0, 6.28, C, 1, 1)) * th.sin())
    for v in _dirs(g, 3):             # a few small suns
        img = img + _uniform(g, 20, 200, C, 1, 1) * torch.exp(((d * v).sum(-1) - 1) / 0.004)[None]
    return img.float().contiguous()


def _fitted(case, seed):
    """Inputs of the inverse problem, mid-way through a descent."""
    s, g = _scene(case, seed), _gen(seed + 1)
    p = torch.randn(case["S"] + 1, 6, generator=g, device="cuda") * torch.tensor([.05] * 3 + [.001] * 3, device="cuda")
    target = s["albedo"] * (2.0 + s["normals"][:, 2] + 0.2 * s["cotangent"])
    return s, p, target


def _mesh(case, seed):
    """A figure of ellipsoids as one triangle mesh, its vertices' radiance, a camera and an image cotangent."""
    r = np.random.default_rng(seed)
    M, R, G, size = case["parts"], case["rings"], case["segments"], case["size"]
    th = (np.arange(R) + 0.5) / R * np.pi
    ph = np.arange(G) / G * 2 * np.pi
    unit = np.stack([np.sin(th)[:, None] * np.cos(ph), np.sin(th)[:, None] * np.sin(ph),
                     np.cos(th)[:, None] + 0 * ph], -1).reshape(-1, 3)
    i, j = np.meshgrid(np.arange(R - 1), np.arange(G), indexing="ij")
    a, b = (i * G + j).ravel(), (i * G + (j + 1) % G).ravel()
    f = np.concatenate([np.stack([a, b, b + G], 1), np.stack([a, b + G, a + G], 1)])
    c = r.uniform(-1, 1, (M, 3)) * np.array([0.45, 0.3, 0.8])
    ax = r.uniform(0.05, 0.22, (M, 3))
    v = (c[:, None] + ax[:, None] * unit[None]).reshape(-1, 3).astype(np.float32)
    faces = (f[None] + (np.arange(M) * R * G)[:, None, None]).reshape(-1, 3).astype(np.int32)
    fl = 0.45 * size * 4.0
    cam = np.array([[-fl, -size / 2, 0, 4 * size / 2], [0, -size / 2, -fl, 4 * size / 2], [0, -1, 0, 4]], np.float32)
    rad = r.uniform(0.0, 2.0, len(v)).astype(np.float32)
    return v, faces, rad, cam, r.standard_normal((size, size)).astype(np.float32)


# ------------------------------------------------------------------ the program around the call

class _Graph:
    """A captured batched step, given back with the state that holds it."""

    def __init__(self, grid, scenes):
        self.handle = _lib.shv_graph_create(grid, scenes)

    def __del__(self):
        _lib.shv_graph_destroy(self.handle)


def _prepare_batch(case, seed):
    subs = _batch_cases(case)
    P, S, N = (sum(f(c) for c in subs) for f in (lambda c: c["P"], lambda c: c["S"], lambda c: c["n"] ** 2))
    out = dict(radiance=torch.empty(P, device="cuda"), grad_points=torch.empty(3 * P, device="cuda"),
               grad_normals=torch.empty(3 * P, device="cuda"), grad_albedo=torch.empty(P, device="cuda"),
               grad_spheres=torch.empty(4 * S, device="cuda"), grad_light=torch.empty(N, device="cuda"))
    at = dict.fromkeys(out, 0)
    bufs, recs = [], []
    for i, c in enumerate(subs):
        s = _scene(c, seed * 64 + i)
        b = batch.SceneBuffers(points=s["points"].t().contiguous(), normals=s["normals"].t().contiguous(),
                               albedo=s["albedo"], spheres=s["spheres"], light=s["light"],
                               grad_radiance=s["cotangent"], n_bands=c["n"], eps=EPS, n_squarings=c["k"], grads=())
        b.allocate()
        rec = b.record()
        sizes = dict(radiance=c["P"], grad_points=3 * c["P"], grad_normals=3 * c["P"], grad_albedo=c["P"],
                     grad_spheres=4 * c["S"], grad_light=c["n"] ** 2)
        for name, m in sizes.items():
            setattr(rec, name, out[name][at[name]:].data_ptr())
            at[name] += m
        bufs.append(b)
        recs.append(rec)
    ops.ensure_init(torch.device("cuda", torch.cuda.current_device()))
    table = batch.Table(recs, bufs[0].points.device)
    return dict(bufs=bufs, recs=recs, out=out, graph=_Graph(table.grid, len(recs)))


def prepare(case, seed):
    kind = case["kind"]
    st = dict(case=case)
    if kind in ("shade", "mode", "rgb"):
        s = _rgb(case, seed) if kind == "rgb" else _scene(case, seed)
        names = ("points", "spheres") if kind == "mode" else INPUTS
        st["inputs"] = [s[k].requires_grad_(True) for k in names]
        st["cotangent"] = s["cotangent"]
        if kind == "mode":
            st["cotangent"] = torch.randn(case["P"], case["n"] ** 2, generator=_gen(seed + 1), device="cuda")
    elif kind in ("render", "forward"):
        s, P, S, N = _scene(case, seed), case["P"], case["S"], case["n"] ** 2
        dev = s["points"].device
        ops.ensure_init(torch.device("cuda", torch.cuda.current_device()))
        prm = _lib.params(case["n"], EPS, case["k"])
        e = lambda *shape: torch.empty(*shape, device=dev)  # noqa: E731
        st.update(prm=prm, pts=s["points"].t().contiguous(), nrm=s["normals"].t().contiguous(), alb=s["albedo"],
                  sph=s["spheres"], light=s["light"], cot=s["cotangent"], vis=e(N, P), rad=e(P),
                  ws=torch.empty(_lib.shv_workspace_bytes(P, S, prm), dtype=torch.uint8, device=dev))
        if kind == "render":
            st.update(saved=e(_lib.shv_render_saved_floats(P, prm)), gP=e(3, P), gN=e(3, P), gA=e(P), gS=e(S, 4),
                      gL=e(N))
    elif kind == "batch":
        st.update(_prepare_batch(case, seed))
    elif kind == "envmap":
        st["image"] = _image(case, seed)
    elif kind == "inverse":
        s, p, target = _fitted(case, seed)
        graph = inverse.DeformGraph(s["points"], s["normals"], s["spheres"], case["K"])
        st.update(p=p, ip=inverse.InverseProblem(graph, s["albedo"], s["light"], target, case["n"], init=p,
                                                 n_squarings=case["k"]))
    else:
        v, faces, rad, cam, gI = _mesh(case, seed)
        V, T, size = len(v), len(faces), case["size"]
        ptr, idx = np.zeros(V + 1, np.int32), np.zeros(3 * T, np.int32)
        _lib.shv_raster_incidence_build(faces, T, V, ptr, idx)
        t = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()  # noqa: E731
        ops.ensure_init(torch.device("cuda", torch.cuda.current_device()))
        st.update(v=t(v.T), faces=t(faces), rad=t(rad), gI=t(gI), ptr=t(ptr), idx=t(idx), V=V, T=T,
                  cam=_lib.camera(cam, size, size), image=torch.empty(size, size, device="cuda"),
                  face_id=torch.empty(size, size, dtype=torch.int32, device="cuda"),
                  gR=torch.empty(V, device="cuda"), gV=torch.empty(3, V, device="cuda"),
                  ws=torch.empty(_lib.shv_raster_workspace_bytes(V, T, size, size), dtype=torch.uint8, device="cuda"))
    return st


def run(st):
    c = st["case"]
    kind = c["kind"]
    if kind in ("shade", "rgb", "mode"):
        x = st["inputs"]
        if kind == "shade":
            y = ops.shade_sh(*x, c["n"], EPS, c["k"])
        elif kind == "rgb":
            y = ops.shade_sh_channels(*x, c["n"], EPS, c["k"])
        else:
            y = ops.visibility_sh(*x, c["n"], EPS, c["k"], mode=c["mode"])
        return [y.detach(), *torch.autograd.grad(y, x, st["cotangent"])]
    stream = torch.cuda.current_stream().cuda_stream
    if kind in ("render", "forward"):
        prm, P, S, ws, saved = st["prm"], c["P"], c["S"], st["ws"], st.get("saved")
        _lib.sh_render_forward(st["pts"], st["nrm"], st["alb"], st["sph"], st["light"], P, S, prm, st["vis"],
                               st["rad"], saved, _lib.nbytes(saved), ws, ws.numel(), stream)
        if kind == "forward":
            return [st["vis"], st["rad"]]
        _lib.sh_render_backward(st["cot"], st["pts"], st["nrm"], st["alb"], st["sph"], P, S, prm, st["vis"], saved,
                                _lib.nbytes(saved), st["gP"], st["gN"], st["gA"], st["gS"], st["gL"], ws, ws.numel(),
                                stream)
        return [st["vis"], st["rad"], st["gP"], st["gN"], st["gA"], st["gS"], st["gL"]]
    if kind == "batch":
        _lib.shv_graph_launch(st["graph"].handle, st["recs"], stream)
        return st["out"]
    if kind == "envmap":
        return ops.envmap_to_sh(st["image"], c["n"])
    if kind == "inverse":
        ip = st["ip"]
        ip.params.copy_(st["p"])
        ip.step()
        return [ip.rad, ip.loss, ip.grad, ip.params]
    cam, ws, V, T = st["cam"], st["ws"], st["V"], st["T"]
    _lib.sh_raster_forward(st["v"], V, st["faces"], T, st["rad"], cam, st["image"], st["face_id"], ws, ws.numel(),
                           stream)
    _lib.sh_raster_backward(st["gI"], st["v"], V, st["faces"], T, st["rad"], cam, st["face_id"], st["ptr"], st["idx"],
                            st["gR"], st["gV"], ws, ws.numel(), stream)
    return [st["image"], st["face_id"], st["gR"], st["gV"]]


# ------------------------------------------------------------------ what a pass cannot do without

def _product_flops(n):
    """One truncated product of two n-band functions, through the smallest exact set of latitudes."""
    lat = (3 * n - 1) // 2
    return 2 * lat * (3 * n * n + 2 * n * n)


def work(case):
    kind = case["kind"]
    if kind == "batch":
        each = [work(c) for c in _batch_cases(case)]
        return {k: sum(w[k] - (c["P"] * c["n"] ** 2 * 4 if k == "bytes" else 0) for w, c in
                       zip(each, _batch_cases(case))) for k in ("bytes", "flops")}
    n = case.get("n", 0)
    N = n * n
    if kind == "envmap":
        px = case["H"] * case["W"] * case["C"]
        return {"bytes": 4 * (px + case["C"] * N), "flops": 2 * N * px}
    if kind == "raster":
        V, px = case["parts"] * case["rings"] * case["segments"], case["size"] ** 2
        T = 2 * case["parts"] * (case["rings"] - 1) * case["segments"]
        return {"bytes": 4 * (2 * 4 * V + 2 * 3 * T + 3 * px), "flops": 60 * T + 60 * px}
    P, S, C, k = case["P"], case["S"], case.get("C", 1), case["k"]
    pair, prod = 5 * N, _product_flops(n)
    back = kind != "forward"
    if kind == "mode" and case["mode"] == "product":
        flops = P * S * (pair + prod + 12 * N + 2 * prod)
    elif kind == "mode" and case["mode"] == "quadrature":
        grid = 32 * n * n
        flops = P * S * (pair + 12 * N) + P * 5 * (grid * 2 * n + grid)
    else:
        more = int(case["mode"][6:]) if kind == "mode" else 0
        flops = P * (S * (pair + (12 * N if back else 0)) + (k + more) * prod * (3 if back else 1))
        flops += 0 if kind == "mode" else P * C * 2 * N * N * (2 if back else 1)
    values = P * (6 + C + N + C) + 4 * S + C * N
    if back:
        values += P * (C + 6 + C) + 4 * S + C * N
    if kind == "mode":
        values = P * (3 + 2 * N + 3) + 8 * S
    if kind == "inverse":
        values, flops = values + P * 12 + S * case["K"] * 4 + 18 * S, flops + S * case["K"] * 200
    if kind in ("shade", "rgb", "inverse"):
        values -= P * N                       # the visibility stays inside the call
    return {"bytes": 4 * values, "flops": flops}


# ------------------------------------------------------------------ the same outputs in 64 bits

def _legendre_sh(d, n):
    """Real orthonormal spherical harmonics of unit directions [..., 3] -> [..., n^2] (no Condon-Shortley phase)."""
    x, y, z = d.unbind(-1)
    cm, sm = [torch.ones_like(x)], [torch.zeros_like(x)]
    for m in range(1, n):
        cm.append(cm[-1] * x - sm[-1] * y)
        sm.append(sm[-1] * x + cm[m - 1] * y)
    out = [None] * (n * n)
    for m in range(n):
        prev, cur = None, torch.full_like(z, math.sqrt((2 * m + 1) / (4 * math.pi) * math.prod(
            (2 * i - 1) / (2 * i) for i in range(1, m + 1))))
        for l in range(m, n):
            if l > m:
                a = math.sqrt((4 * l * l - 1) / (l * l - m * m))
                b = math.sqrt(((l - 1) ** 2 - m * m) / (4 * (l - 1) ** 2 - 1)) if l > m + 1 else 0.0
                prev, cur = cur, a * (z * cur - (b * prev if l > m + 1 else 0.0))
            if m == 0:
                out[l * l + l] = cur
            else:
                out[l * l + l + m] = math.sqrt(2) * cur * cm[m]
                out[l * l + l - m] = math.sqrt(2) * cur * sm[m]
    return torch.stack(out, -1)


def _rule(degree, n):
    """Nodes' harmonics [Q, n^2] and weights [Q] of a product rule exact to ``degree``."""
    z, w = np.polynomial.legendre.leggauss(degree // 2 + 1)
    m = degree + 1
    ph = (np.arange(m) + 0.5) * 2 * np.pi / m
    r = np.sqrt(1 - z * z)
    d = np.stack([r[:, None] * np.cos(ph), r[:, None] * np.sin(ph), z[:, None] + 0 * ph], -1).reshape(-1, 3)
    t = torch.as_tensor(d, device="cuda")
    return _legendre_sh(t, n), torch.as_tensor(np.repeat(w * 2 * np.pi / m, m), device="cuda")


def _band(n):
    return torch.tensor([math.isqrt(i) for i in range(n * n)], device="cuda")


def _cap(t, n):
    """2 pi int_t^1 P_l for l < n -> [..., n]."""
    p = [torch.ones_like(t), t]
    for l in range(2, n + 1):
        p.append(((2 * l - 1) * t * p[-1] - (l - 1) * p[-2]) / l)
    return torch.stack([2 * math.pi * ((1 - t) if l == 0 else (p[l - 1] - p[l + 1]) / (2 * l + 1))
                        for l in range(n)], -1)


def _caps(points, spheres, n):
    """Cap integrals [P, S, n], harmonics of the spheres' directions [P, S, n^2]."""
    v = spheres[None, :, :3] - points[:, None]
    d = v.norm(dim=-1)
    u = 1 - (spheres[None, :, 3] / d) ** 2
    t = torch.where(u > 0, u.clamp(min=1e-300).sqrt(), torch.zeros_like(u))
    return _cap(t, n), _legendre_sh(v / d[..., None], n)


def _visibility(points, spheres, n, k, mode="squaring"):
    band = _band(n)
    caps, Y = _caps(points, spheres, n)
    Yq, w = _rule(3 * n - 3, n)

    def product(a, b):
        return ((a @ Yq.T) * (b @ Yq.T) * w) @ Yq

    if mode == "product":
        full = torch.zeros(n, dtype=F64, device="cuda")
        full[0] = 4 * math.pi
        b = (full + math.expm1(-EPS) * caps)[..., band] * Y
        V = torch.zeros(points.shape[0], n * n, dtype=F64, device="cuda")
        V[:, 0] = SQRT_4PI
        for i in range(spheres.shape[0]):
            V = product(V, b[:, i])
        return V
    F = (-EPS * caps[..., band] * Y).sum(1)
    c = F[:, :1] / SQRT_4PI
    G = torch.cat([torch.zeros_like(c), F[:, 1:]], 1)
    if mode == "quadrature":
        Yr, wr = _rule(8 * n - 1, n)
        return torch.exp(c) * ((torch.exp(G @ Yr.T) * wr) @ Yr)
    G = G * 2.0 ** -k
    one = torch.zeros(n * n, dtype=F64, device="cuda")
    one[0] = SQRT_4PI
    if mode == "squaring":
        E = torch.exp((G * G).sum(1, keepdim=True) / (8 * math.pi)) * (one + G)
    else:
        E, power = one + G, G
        for j in range(2, int(mode[6:]) + 1):
            power = product(power, G)
            E = E + power / math.factorial(j)
    for _ in range(k):
        E = product(E, E)
    return torch.exp(c) * E


def _shade(V, normals, albedo, light, n):
    """a_c (L_c . (V * H)) for albedo [P, C], light [C, N]."""
    zs, ws = np.polynomial.legendre.leggauss(2 * n)
    x, wx = (zs + 1) / 2, ws / 2
    A = []
    for l in range(n):
        c = np.zeros(l + 1)
        c[l] = 1
        A.append(2 * math.pi * float((wx * x * np.polynomial.legendre.legval(x, c)).sum()))
    H = torch.tensor(A, dtype=F64, device="cuda")[_band(n)] * _legendre_sh(normals / normals.norm(dim=1, keepdim=True), n)
    Yq, w = _rule(3 * n - 3, n)
    return albedo * (((V @ Yq.T) * (H @ Yq.T) * w) @ (light @ Yq.T).T)


def _chunks(P, S, n, room):
    m = max(64, room // max(1, S * n * n))
    return [slice(a, min(P, a + m)) for a in range(0, P, m)]


def _exact_render(s, case, back=True):
    """V, B and the gradients to the inputs of one scene, chunk by chunk over receivers."""
    n, k, P = case["n"], case["k"], s["points"].shape[0]
    d = {key: v.double() for key, v in s.items()}
    mono = d["albedo"].dim() == 1
    if mono:
        d["albedo"], d["light"], d["cotangent"] = d["albedo"][:, None], d["light"][None], d["cotangent"][:, None]
    V, B, g = [], [], {key: [] for key in INPUTS}
    for sl in _chunks(P, d["spheres"].shape[0], n, 48_000_000):
        x = [d["points"][sl], d["normals"][sl], d["albedo"][sl], d["spheres"], d["light"]]
        x = [t.clone().requires_grad_(back) for t in x]
        with torch.set_grad_enabled(back):
            v = _visibility(x[0], x[3], n, k)
            b = _shade(v, x[1], x[2], x[4], n)
            if back:
                for key, t in zip(INPUTS, torch.autograd.grad(b, x, d["cotangent"][sl])):
                    g[key].append(t)
        V.append(v.detach())
        B.append(b.detach())
    out = [torch.cat(V), torch.cat(B)]
    if back:
        out += [torch.cat(g[key]) for key in INPUTS[:3]] + [sum(g["spheres"]), sum(g["light"])]
    if mono:
        out[1] = out[1][:, 0]
        if back:
            out[4], out[6] = out[4][:, 0], out[6][0]
    return out


def _rotations(a):
    """Rodrigues' matrices of axis-angle vectors [M, 3]."""
    t2 = (a * a).sum(-1)
    t = t2.clamp(min=1e-24).sqrt()
    A, B = torch.sin(t) / t, (torch.sin(t / 2) / t) ** 2 * 2
    z = torch.zeros_like(t)
    K = torch.stack([z, -a[:, 2], a[:, 1], a[:, 2], z, -a[:, 0], -a[:, 1], a[:, 0], z], -1).view(-1, 3, 3)
    return torch.eye(3, dtype=F64, device="cuda") + A[:, None, None] * K + B[:, None, None] * (K @ K)


def _exact_inverse(case, seed):
    s, p, target = _fitted(case, seed)
    d = {key: v.double() for key, v in s.items()}
    P, S, K = case["P"], case["S"], case["K"]
    v, m, g = d["points"], d["normals"], d["spheres"][:, :3]
    near = torch.stack([((v - c) ** 2).sum(1) for c in g])
    dist, idx = torch.sort(near, dim=1, stable=True)
    top = dist[:, min(K, P - 1)].sqrt()
    u = (1 - dist[:, :K].sqrt() / top[:, None]) ** 2
    idx = idx[:, :K]
    tot = torch.zeros(P, dtype=F64, device="cuda").index_add_(0, idx.reshape(-1), u.reshape(-1))
    w = torch.where(tot[idx] > 0, u / tot[idx], torch.zeros_like(u))
    rest = 1 - torch.zeros(P, dtype=F64, device="cuda").index_add_(0, idx.reshape(-1), w.reshape(-1))
    p = p.double().requires_grad_(True)
    R = _rotations(p[:, :3])
    loc = ((v[idx] - g[:, None])[:, :, None, :] * R[:S, None]).sum(-1) + (g + p[:S, 3:])[:, None]
    nloc = (m[idx][:, :, None, :] * R[:S, None]).sum(-1)
    y = (rest[:, None] * v).index_add(0, idx.reshape(-1), (w[..., None] * loc).reshape(-1, 3))
    z = (rest[:, None] * m).index_add(0, idx.reshape(-1), (w[..., None] * nloc).reshape(-1, 3))
    x, nr = y @ R[S].T + p[S, 3:], z @ R[S].T
    sph = torch.cat([(g + p[:S, 3:]) @ R[S].T + p[S, 3:], d["spheres"][:, 3:]], 1)
    now = dict(points=x.detach(), normals=nr.detach(), albedo=d["albedo"], spheres=sph.detach(), light=d["light"],
               cotangent=d["cotangent"])
    B = _exact_render(now, case, back=False)[1]
    now["cotangent"] = 2 * (B - target.double()) / P
    o = _exact_render(now, case)
    grad = torch.autograd.grad([x, nr, sph], p, [o[2], o[3], o[5]])[0]
    return [B, ((B - target.double()) ** 2).mean()[None], grad, p.detach() - 1e-2 * grad]


def _exact_raster(case, seed):
    """Faces by the library's stated single-precision decisions (one rounding an operation), values in 64 bits."""
    v, faces, rad, cam, gI = _mesh(case, seed)
    size, f32 = case["size"], np.float32
    x, y, z = v.T
    u, q, w = (((c[0] * x + c[1] * y) + c[2] * z) + c[3] for c in cam)
    X, Y, W = (u / w)[faces], (q / w)[faces], w[faces]
    area = (X[:, 1] - X[:, 0]) * (Y[:, 2] - Y[:, 0]) - (X[:, 2] - X[:, 0]) * (Y[:, 1] - Y[:, 0])
    ok = (W > f32(1e-6)).all(1) & (area != 0) & np.isfinite(area)
    i0 = np.maximum(np.floor(X.min(1) - 0.5), 0).astype(np.int64)
    i1 = np.minimum(np.ceil(X.max(1) - 0.5), size - 1).astype(np.int64)
    j0 = np.maximum(np.floor(Y.min(1) - 0.5), 0).astype(np.int64)
    j1 = np.minimum(np.ceil(Y.max(1) - 0.5), size - 1).astype(np.int64)
    best = np.full(size * size, np.iinfo(np.int64).max)
    for dj in range(int((j1 - j0).max(initial=0)) + 1):
        for di in range(int((i1 - i0).max(initial=0)) + 1):
            t = np.nonzero(ok & (i0 + di <= i1) & (j0 + dj <= j1))[0]
            px, py = (i0[t] + di).astype(f32) + f32(0.5), (j0[t] + dj).astype(f32) + f32(0.5)
            xs, ys, ws = X[t].T, Y[t].T, W[t].T
            lam = [((xs[a] - px) * (ys[b] - py) - (xs[b] - px) * (ys[a] - py)) / area[t]
                   for a, b in ((1, 2), (2, 0), (0, 1))]
            zz = f32(1) / ((lam[0] / ws[0] + lam[1] / ws[1]) + lam[2] / ws[2])
            hit = (lam[0] >= 0) & (lam[1] >= 0) & (lam[2] >= 0)
            key = (zz[hit].view(np.int32).astype(np.int64) << 32) | t[hit]
            np.minimum.at(best, (j0[t] + dj)[hit] * size + (i0[t] + di)[hit], key)
    face = np.where(best == np.iinfo(np.int64).max, -1, best & 0xFFFFFFFF)
    at = np.nonzero(face >= 0)[0]
    vt, rt = torch.tensor(v.T, dtype=F64, requires_grad=True), torch.tensor(rad, dtype=F64, requires_grad=True)
    cm = torch.tensor(cam, dtype=F64)
    h = cm[:, :3] @ vt + cm[:, 3:]
    f = torch.as_tensor(faces[face[at]].astype(np.int64))
    xs, ys, ws = (h[0] / h[2])[f], (h[1] / h[2])[f], h[2][f]
    px, py = torch.as_tensor(at % size + 0.5), torch.as_tensor(at // size + 0.5)
    lam = torch.stack([(xs[:, a] - px) * (ys[:, b] - py) - (xs[:, b] - px) * (ys[:, a] - py)
                       for a, b in ((1, 2), (2, 0), (0, 1))], 1) / ws
    img = torch.zeros(size * size, dtype=F64).index_put((torch.as_tensor(at),),
                                                        (lam * rt[f]).sum(1) / lam.sum(1))
    gR, gV = torch.autograd.grad(img, [rt, vt], torch.as_tensor(gI.reshape(-1)).double())
    return [img.detach().view(size, size), torch.as_tensor(face.reshape(size, size)).int(), gR, gV]


def exact(case, seed):
    kind = case["kind"]
    if kind == "shade":
        return _exact_render(_scene(case, seed), case)[1:]
    if kind == "rgb":
        return _exact_render(_rgb(case, seed), case)[1:]
    if kind == "forward":
        V, B = _exact_render(_scene(case, seed), case, back=False)
        return [V.t(), B]
    if kind == "render":
        V, B, gP, gN, *rest = _exact_render(_scene(case, seed), case)
        return [V.t(), B, gP.t(), gN.t(), *rest]
    if kind == "batch":
        outs = [_exact_render(_scene(c, seed * 64 + i), c)[1:] for i, c in enumerate(_batch_cases(case))]
        names = ("radiance", "grad_points", "grad_normals", "grad_albedo", "grad_spheres", "grad_light")
        return {m: torch.cat([(o[j].t() if j in (1, 2) else o[j]).reshape(-1) for o in outs])
                for j, m in enumerate(names)}
    if kind == "mode":
        s, n = _scene(case, seed), case["n"]
        cot = torch.randn(case["P"], n * n, generator=_gen(seed + 1), device="cuda").double()
        nodes = 32 * n * n if case["mode"] == "quadrature" else 8 * n * n * case["S"]
        V, gp, gs = [], [], 0
        for sl in _chunks(case["P"], case["S"] + nodes // (n * n), n, 96_000_000):
            x = [s["points"][sl].double().requires_grad_(True), s["spheres"].double().requires_grad_(True)]
            v = _visibility(*x, n, case["k"], case["mode"])
            a, b = torch.autograd.grad(v, x, cot[sl])
            V.append(v.detach())
            gp.append(a)
            gs = gs + b
        return [torch.cat(V), torch.cat(gp), gs]
    if kind == "envmap":
        img, n, H, W = _image(case, seed).double(), case["n"], case["H"], case["W"]
        th = (torch.arange(H, device="cuda", dtype=F64) + 0.5) * math.pi / H
        ph = (torch.arange(W, device="cuda", dtype=F64) + 0.5) * 2 * math.pi / W
        edge = torch.cos(torch.arange(H + 1, device="cuda", dtype=F64) * math.pi / H)
        omega = (edge[:-1] - edge[1:]) * 2 * math.pi / W
        L = 0
        for a in range(0, H, 64):
            t = th[a:a + 64, None]
            d = torch.stack([t.sin() * ph.cos(), t.sin() * ph.sin(), t.cos() + 0 * ph], -1)
            L = L + (img[:, a:a + 64] * omega[a:a + 64, None]).reshape(case["C"], -1) @ _legendre_sh(d, n).view(-1, n * n)
        return L
    if kind == "inverse":
        return _exact_inverse(case, seed)
    return _exact_raster(case, seed)
