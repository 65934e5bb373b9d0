"""Performance cases of the estimator, through its public Python entry points.

A case is a dict of plain values.  Kinds of case:

  step      Context.estimate_grad into kept accumulators, then Context.step
            (the optimisation loop that a program writes itself)
  batch     Batch.step, replayed as a graph (one scene, or many uneven ones)
  grad      Context.estimate_grad into new accumulators, then decode_grad
            (the gradient for another optimiser); `form` picks the per-pixel
            loss form, the full-image estimator, the image form or the
            allocation-free call
  autograd  StochasticRender / StochasticRasterLoss, forward and backward
  render    Context.render of every view: colours, IDs and UVs

Scenes are geodesic spheres with perturbed vertices and textures in the
middle of an optimisation, Catmull-Clark control spheres, or triangle soups;
sizes are those of scenes.py and bench.py, and ragged ones between them.
Learning rates are a fiftieth of the perturbation, as late in a run whose
rate has decayed, so that a state keeps its character over many passes.
"""
import functools
import math

import numpy as np
import torch
import torch.nn.functional as F

from paper_2404_09758_amd import api, autograd, batch, scenes

DEV = "cuda:0"
LR_OF_EPS = 0.02
SPHERE_COVER = 0.57      # share of the pixels that a unit sphere covers at the scenes' camera


def _case(name, kind, **kw):
    c = {"name": name, "kind": kind, "mesh": "sphere", "freq": 32, "splits": 0, "width": 512, "height": 512,
         "tex_w": 512, "tex_h": 512, "shading": 1, "layers": 0, "subdiv": 0, "views": 1, "pairs": 1, "tile": 16,
         "items": 0, "optimizer": "adam", "form": "loss", "scenes": 1}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: the 64 px, 320-triangle scene, one pair, SGD; launches and host time count
        _case("tiny_step", "step", freq=4, width=64, height=64, tex_w=64, tex_h=64, shading=0, items=1,
              optimizer="sgd"),
        # the 512 px Lambert workload, 8 ring views x 16 pairs, with the Context's default launch shape
        # (one raster launch per pair and view)
        _case("mid_step_plain", "step", views=8, pairs=16, items=1),
        # the paper-scale step written as a loop over one Context: 1024 px, 46080 triangles, GGX, three maps
        _case("paper_step", "step", freq=12, splits=2, width=1024, height=1024, tex_w=1024, tex_h=1024, shading=2,
              views=4, pairs=8),
        # the same step as a captured graph, the form of the headline benchmark
        _case("paper_graph", "batch", freq=12, splits=2, width=1024, height=1024, tex_w=1024, tex_h=1024, shading=2,
              views=4, pairs=8),
        # many independent scenes of uneven size stepped together
        _case("batch_12_scenes", "batch", scenes=12, pairs=4, width=1024, height=1024, tex_w=1024, tex_h=1024,
              freq=48),
        # semi-transparent geometry: two nearest layers
        _case("layers_2_step", "step", layers=2, views=4, pairs=8),
        # four layers, ragged image and texture, gradient of a downstream loss
        _case("layers_4_ragged_grad", "grad", layers=4, views=3, pairs=4, width=501, height=333, tex_w=300,
              tex_h=213, freq=21, form="image"),
        # subdivision surface: 2000 control triangles, two levels, GGX
        _case("subdiv_step", "step", subdiv=2, freq=10, width=1024, height=1024, tex_w=1024, tex_h=1024, shading=2,
              views=4, pairs=8),
        # triangle soup of the per-pixel against full-image comparison, 128 pairs, nearest texels
        _case("soup_10k_step", "step", mesh="soup", freq=10240, shading=0, pairs=128),
        # the full-image estimator on the same soup
        _case("soup_10k_full", "grad", mesh="soup", freq=10240, shading=0, pairs=128, form="full"),
        # the render as a differentiable function in a torch program, ragged sizes
        _case("autograd_ragged", "autograd", width=500, height=333, tex_w=300, tex_h=200, freq=20, views=3, pairs=16,
              form="image"),
        # forward only: looking at the scene, with its ID and UV buffers
        _case("render_1024", "render", freq=12, splits=2, width=1024, height=1024, tex_w=1024, tex_h=1024, shading=2,
              views=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "batch", "grad", "grad", "autograd", "render"])
    w, h = _log_int(rng, 48, 1024), _log_int(rng, 48, 1024)
    c = _case("", kind, width=w, height=h, tex_w=_log_int(rng, 32, 1024), tex_h=_log_int(rng, 32, 1024),
              freq=_log_int(rng, 4, 45), shading=rng.choice([0, 1, 1, 2]), views=rng.randint(1, 6),
              pairs=_log_int(rng, 1, 32), tile=rng.choice([8, 16, 16, 16, 32]), items=rng.choice([0, 0, 1]),
              optimizer=rng.choice(["adam", "adam", "sgd"]))
    del c["name"]
    what = rng.choice(["sphere", "sphere", "sphere", "layers", "subdiv", "soup"])
    if kind == "batch":
        c["scenes"] = rng.choice([1, 2, 5, 9])
        c["items"] = 0
    elif kind == "autograd":
        c["shading"] = min(c["shading"], 1)
        c["form"] = rng.choice(["image", "loss"])
    elif kind == "grad":
        c["form"] = rng.choice(["loss", "image", "full", "noalloc"])
    cost = 1.0
    if kind in ("step", "grad", "render"):
        if what == "layers":
            c["layers"], c["shading"], c["tile"] = rng.randint(1, 4), min(c["shading"], 1), rng.choice([8, 16])
            cost = 4.0 * c["layers"]
        elif what == "subdiv":
            c["subdiv"], c["freq"] = rng.choice([1, 2]), rng.randint(3, 10)
            cost = 2.0
        elif what == "soup":
            c["mesh"], c["freq"], c["shading"], c["views"] = "soup", _log_int(rng, 200, 20000), 0, 1
            c["height"] = c["width"]
            cost = 2.0
    if c["form"] == "noalloc":                       # its scratch is 128 MiB
        c["width"], c["height"], c["freq"] = min(c["width"], 400), min(c["height"], 400), min(c["freq"], 12)
        c["tex_w"], c["tex_h"], c["pairs"] = min(c["tex_w"], 256), min(c["tex_h"], 256), min(c["pairs"], 8)
    limit = 24e6 / cost / c["scenes"]
    c["pairs"] = max(1, min(c["pairs"], int(limit / (c["width"] * c["height"] * c["views"]))))
    return c


# ------------------------------------------------------------------ inputs --

@functools.lru_cache(maxsize=None)
def _mesh(freq, splits):
    v, f = scenes.geodesic_icosphere(freq)
    for _ in range(splits):
        v, f = scenes.midpoint_split(v, f)
    return v, f, scenes.spherical_corner_uv(v, f)


def _waves(v, rng, amp):
    """Smooth radial displacement: a few plane waves of random direction."""
    d = v / np.linalg.norm(v, axis=1, keepdims=True)
    s = np.zeros(len(v))
    for k in range(8):
        s += np.sin(d @ (rng.normal(size=3) * (1.5 + k)) + rng.uniform(0, 6.28)) / (1.5 + k)
    return (v * (1.0 + amp * s)[:, None]).astype(np.float32)


def _image(gen, h, w, c, lo=0.1, hi=0.9):
    """Smooth random field with some fine detail, [h, w, c] on the GPU."""
    g = torch.rand((1, c, max(2, h // 24), max(2, w // 24)), generator=gen, device=DEV)
    t = F.interpolate(g, size=(h, w), mode="bilinear", align_corners=False)[0].permute(1, 2, 0)
    t = 0.85 * t + 0.15 * torch.rand((h, w, c), generator=gen, device=DEV)
    return (lo + (hi - lo) * t).contiguous()


def _textures(case, gen):
    h, w = case["tex_h"], case["tex_w"]
    if case["shading"] != 2:
        return [_image(gen, h, w, 4 if case["layers"] else 3)]
    nrm = torch.stack([0.35 + 0.3 * _image(gen, h, w, 1)[..., 0], 0.35 + 0.3 * _image(gen, h, w, 1)[..., 0],
                       torch.full((h, w), 0.95, device=DEV)], dim=2)
    return [_image(gen, h, w, 3), nrm, _image(gen, h, w, 1, 0.2, 0.8)]


def _scene(case, seed, index=0):
    """The scene's arrays (start and target parameters) from the seed."""
    rng = np.random.default_rng([int(seed), index])
    if case["mesh"] == "soup":
        sc = scenes.make_soup(case["freq"], res=case["width"], seed=int(seed) % 100003, pairs=case["pairs"])
        gen = torch.Generator(device=DEV).manual_seed(int(seed))
        sc.target_image = _image(gen, case["height"], case["width"], 3)
        return sc
    gen = torch.Generator(device=DEV).manual_seed(int(seed) * 64 + index)
    v, f, uv = _mesh(case["freq"], case["splits"])
    tex = [t.cpu().numpy() for t in _textures(case, gen)]
    target = [t.cpu().numpy() for t in _textures(case, gen)]
    eps_pos = 1.5 * (scenes.CAM_DIST * math.tan(math.radians(scenes.FOVY_DEG) / 2)) * 2.0 / max(case["height"], 256)
    n = case["views"]
    az, el = float(rng.uniform(0.0, 360.0)), float(rng.uniform(-25.0, 25.0))
    views = [scenes.look_at_view(case["width"], case["height"], az + 360.0 * k / n, el) for k in range(n)]
    eps = [eps_pos] + [1.0 / 255.0] * len(tex)
    return scenes.Scene("case", f.astype(np.int32), uv, _waves(v, rng, 0.02), tex, _waves(v, rng, 0.05), target, views,
                        shading=case["shading"], ambient=0.03 if case["shading"] == 2 else 0.1,
                        light_rgb=np.full(3, 3.0 if case["shading"] == 2 else 1.0, np.float32), eps=eps,
                        lr=[LR_OF_EPS * e for e in eps], n_pairs=case["pairs"], seed=int(seed) % 100003,
                        layers=case["layers"], subdiv_levels=case["subdiv"])


def _batch_cases(case):
    """Sizes of a batch's scenes: the case's own, then smaller ones, as uneven as scenes.make_batch_scene."""
    r = np.random.default_rng(6)
    out = [case]
    for _ in range(case["scenes"] - 1):
        c = dict(case)
        c["freq"] = max(3, int(case["freq"] * math.exp(r.uniform(math.log(0.15), 0.0))))
        c["width"] = max(40, case["width"] // int(r.choice([1, 2, 4, 8])))
        c["height"] = max(40, case["height"] // int(r.choice([1, 2, 4, 8])))
        c["tex_w"] = c["tex_h"] = max(16, case["tex_w"] // int(r.choice([1, 2, 4, 8])))
        out.append(c)
    return out


def _targets(ctx, sc):
    if hasattr(sc, "target_image"):
        return sc.target_image.reshape(-1).contiguous()
    th = torch.tensor(sc.flat_params(True), device=DEV)
    return torch.cat([ctx.render(th, v, ids=False, uv=False)[0].reshape(-1) for v in sc.views])


def prepare(case, seed):
    s = {"case": case, "t": 0}
    if case["kind"] == "batch":
        scs = [_scene(c, seed, b) for b, c in enumerate(_batch_cases(case))]
        kind = api.ADAM if case["optimizer"] == "adam" else api.SGD
        s["batch"] = batch.Batch(scs, case["pairs"], DEV, tile_px=case["tile"], kind=kind, seed=int(seed) % 100003)
        return s
    sc = _scene(case, seed)
    s["scene"] = sc
    if case["kind"] == "autograd":
        ctx = api.Context(sc, DEV, tuning=(case["tile"], 256, case["items"]))
        kw = {"n_pairs": case["pairs"], "eps": sc.eps[:2], "seed": sc.seed, "device": DEV,
              "tuning": (case["tile"], 256, case["items"])}
        tg = _targets(ctx, sc)
        if case["form"] == "loss":
            s["fn"] = autograd.StochasticRasterLoss(sc, tg, **kw)
        else:
            s["fn"] = autograd.StochasticRender(sc, **kw)
            s["target"] = tg.reshape(len(sc.views), case["height"], case["width"], 3)
        s["pos"] = torch.tensor(sc.pos, device=DEV).requires_grad_()
        s["albedo"] = torch.tensor(sc.tex[0], device=DEV).requires_grad_()
        return s
    s["ctx"] = ctx = api.Context(sc, DEV, tuning=(case["tile"], 256, case["items"]))
    s["theta"] = torch.tensor(sc.flat_params(), device=DEV)
    if case["kind"] == "render":
        return s
    s["target"] = _targets(ctx, sc)
    if case["form"] == "image":
        images = torch.cat([ctx.render(s["theta"], v, ids=False, uv=False)[0].reshape(-1) for v in sc.views])
        s["target"] = 2.0 * (images - s["target"])
    if case["kind"] == "step":
        s["m"], s["v"] = torch.zeros_like(s["theta"]), torch.zeros_like(s["theta"])
        s["Q"], s["K"] = ctx.new_accumulators()
    return s


def run(s):
    case = s["case"]
    if case["kind"] == "batch":
        b = s["batch"]
        b.step(use_graph=True)
        return [b.theta, b.m, b.v]
    sc = s["scene"]
    if case["kind"] == "autograd":
        out = s["fn"](s["pos"], s["albedo"])
        loss = out if case["form"] == "loss" else ((out - s["target"]) ** 2).sum()
        grads = torch.autograd.grad(loss, [s["pos"], s["albedo"]])
        return [out.detach(), list(grads)]
    ctx = s["ctx"]
    if case["kind"] == "render":
        return [list(ctx.render(s["theta"], v)) for v in sc.views]
    s["t"] += 1
    if case["kind"] == "grad":
        Q, K = ctx.estimate_grad(s["theta"], sc.views, s["target"], sc.seed, s["t"], sc.n_pairs, sc.eps,
                                 full_image=case["form"] == "full", image_grad=case["form"] == "image",
                                 noalloc=case["form"] == "noalloc")
        return [Q, K, ctx.decode_grad(Q, K, sc.eps, n_pairs=sc.n_pairs)]
    lr = [LR_OF_EPS * e for e in sc.eps]
    ctx.estimate_grad(s["theta"], sc.views, s["target"], sc.seed, s["t"], sc.n_pairs, sc.eps, Q=s["Q"], K=s["K"])
    ctx.step(s["theta"], s["m"], s["v"], s["t"], s["Q"], s["K"], sc.eps, sc.n_pairs,
             kind=api.ADAM if case["optimizer"] == "adam" else api.SGD, lr=lr)
    return [s["theta"], s["m"], s["v"]]


# -------------------------------------------------------------------- work --

def _sizes(case):
    """(triangles, vertices, parameters, texel groups) of one scene."""
    if case["mesh"] == "soup":
        n = case["freq"]
        return n, 3 * n, 12 * n, n
    n = case["freq"] << case["splits"]
    tris, verts = 20 * n * n, 10 * n * n + 2
    texels = case["tex_w"] * case["tex_h"]
    ch = 7 if case["shading"] == 2 else (4 if case["layers"] else 3)
    if case["subdiv"]:                               # 3 quads per control triangle, 4 per quad, 2 triangles each
        return 6 * tris * 4 ** (case["subdiv"] - 1), verts, 3 * verts + ch * texels, texels
    return tris, verts, 3 * verts + ch * texels, texels


def _work_one(case):
    tris, verts, d, texels = _sizes(case)
    px = case["width"] * case["height"] * case["views"]
    est = case["kind"] != "render"
    renders = 2 * case["pairs"] if est else 1
    shade = (82, 85, 300)[case["shading"]] * max(1, case["layers"])       # operations of one shaded pixel
    covered = px * (1.0 if case["mesh"] == "soup" else SPHERE_COVER)
    flops = renders * (covered * (shade + 22) + tris * case["views"] * 150.0)
    if not est:
        deep = max(1, case["layers"])
        return 4.0 * d + px * (12 + 12 * deep), flops
    flops += covered * case["pairs"] * 25 + 20.0 * d
    groups = verts + texels
    nbytes = 12.0 * px + 8.0 * tris * 3
    if case["kind"] in ("step", "batch"):
        nbytes += (24.0 if case["optimizer"] == "adam" else 8.0) * d
    elif case["kind"] == "grad":
        nbytes += 4.0 * d + 12.0 * d + 4.0 * groups                       # theta in; Q, K and the gradient out
    else:
        nbytes += 8.0 * d + 24.0 * px
    return nbytes, flops


def work(case):
    parts = [_work_one(c) for c in (_batch_cases(case) if case["kind"] == "batch" else [case])]
    return {"bytes": float(sum(p[0] for p in parts)), "flops": float(sum(p[1] for p in parts))}


# ------------------------------------------------------------------- exact --

def _unit(x):
    return x / x.norm(dim=-1, keepdim=True).clamp_min(1e-300)


def _bilinear(tex, u, v):
    """Bilinear sample of [h, w, c]: texel centres at half-integers, u wraps, v clamps."""
    h, w = tex.shape[:2]
    x, y = u * w - 0.5, v * h - 0.5
    x0, y0 = x.floor(), y.floor()
    fx, fy = (x - x0)[:, None], (y - y0)[:, None]
    xa, xb = x0.long() % w, (x0.long() + 1) % w
    ya, yb = y0.long().clamp(0, h - 1), (y0.long() + 1).clamp(0, h - 1)
    return ((1 - fx) * tex[ya, xa] + fx * tex[ya, xb]) * (1 - fy) + ((1 - fx) * tex[yb, xa] + fx * tex[yb, xb]) * fy


def _render64(sc, view):
    """Colours [h, w, 3] and UVs [h, w, 2] of an opaque scene in float64: nearest covering triangle at each
    pixel centre, vertices on the 1/256-pixel grid, perspective-correct attributes, unlit / Lambert / GGX."""
    f8 = {"dtype": torch.float64, "device": DEV}
    W, H = view.width, view.height
    pos, tri = torch.tensor(sc.pos, **f8), torch.tensor(sc.tri, device=DEV).long()
    M = torch.tensor(view.view_proj, **f8)
    clip = torch.cat([pos, torch.ones_like(pos[:, :1])], 1) @ M.T
    ndc = clip[:, :3] / clip[:, 3:]
    sx = torch.round((ndc[:, 0] * 0.5 + 0.5) * W * 256) / 256
    sy = torch.round((0.5 - ndc[:, 1] * 0.5) * H * 256) / 256
    X, Y, Z, iw = sx[tri], sy[tri], (ndc[:, 2] * 0.5 + 0.5)[tri], (1 / clip[:, 3])[tri]
    x0 = (X.amin(1) - 0.5).ceil().clamp(min=0).long()
    x1 = (X.amax(1) - 0.5).floor().clamp(max=W - 1).long()
    y0 = (Y.amin(1) - 0.5).ceil().clamp(min=0).long()
    y1 = (Y.amax(1) - 0.5).floor().clamp(max=H - 1).long()
    bw, bh = (x1 - x0 + 1).clamp(min=0), (y1 - y0 + 1).clamp(min=0)
    n = bw * bh
    t = torch.repeat_interleave(torch.arange(len(tri), device=DEV), n)
    k = torch.arange(len(t), device=DEV) - torch.repeat_interleave(n.cumsum(0) - n, n)
    x, y = x0[t] + k % bw[t], y0[t] + k // bw[t]
    cx, cy = x + 0.5, y + 0.5

    def edge(a, b):
        return (X[t, b] - X[t, a]) * (cy - Y[t, a]) - (Y[t, b] - Y[t, a]) * (cx - X[t, a])
    e = torch.stack([edge(1, 2), edge(2, 0), edge(0, 1)], 1)
    area = e.sum(1, keepdim=True)
    bary = e / torch.where(area == 0, torch.ones_like(area), area)
    ok = (area[:, 0] != 0) & (bary >= 0).all(1)
    t, bary, pix = t[ok], bary[ok], (y * W + x)[ok]
    z = (bary * Z[t]).sum(1)
    zmin = torch.full((H * W,), math.inf, **f8).scatter_reduce(0, pix, z, "amin")
    near = z == zmin[pix]
    t, bary, pix = t[near], bary[near], pix[near]
    first = torch.full((H * W,), len(tri), device=DEV).scatter_reduce(0, pix, t, "amin")
    keep = t == first[pix]
    t, bary, pix = t[keep], bary[keep], pix[keep]
    pc = bary * iw[t]
    pc = pc / pc.sum(1, keepdim=True)
    cuv = torch.tensor(sc.corner_uv, **f8)
    uv = (pc[:, :, None] * cuv[t]).sum(1)
    tex = [torch.tensor(a, **f8) for a in sc.tex]
    alb = _bilinear(tex[0], uv[:, 0], uv[:, 1])[:, :3]
    P3 = pos[tri]
    e1, e2 = P3[:, 1] - P3[:, 0], P3[:, 2] - P3[:, 0]
    N = _unit(torch.linalg.cross(e1, e2))
    L, rgb_l = torch.tensor(sc.light_dir, **f8), torch.tensor(sc.light_rgb, **f8)
    if sc.shading == 0:
        rgb = alb
    elif sc.shading == 1:
        rgb = alb * (sc.ambient + sc.diffuse * (N[t] @ L).clamp(min=0))[:, None] * rgb_l
    else:
        d1, d2 = cuv[:, 1] - cuv[:, 0], cuv[:, 2] - cuv[:, 0]
        T = e1 * d2[:, 1:] - e2 * d1[:, 1:]
        T = torch.where((d1[:, :1] * d2[:, 1:] - d2[:, :1] * d1[:, 1:]) < 0, -T, T)
        T = _unit(T - N * (N * T).sum(1, keepdim=True))
        B = torch.linalg.cross(N, T)
        tn = 2 * _bilinear(tex[1], uv[:, 0], uv[:, 1]) - 1
        nn = _unit(T[t] * tn[:, :1] + B[t] * tn[:, 1:2] + N[t] * tn[:, 2:])
        V = _unit(torch.tensor(view.cam_pos, **f8) - (pc[:, :, None] * P3[t]).sum(1))
        Hh = _unit(L + V)
        ndl, ndv = (nn @ L).clamp(min=0), (nn * V).sum(1).clamp(min=0)
        ndh, vdh = (nn * Hh).sum(1).clamp(min=0), (V * Hh).sum(1).clamp(min=0)
        al = (_bilinear(tex[2], uv[:, 0], uv[:, 1])[:, 0] ** 2).clamp(min=0.002)
        a2, kk = al * al, al / 2
        dd = ndh * ndh * (a2 - 1) + 1
        Fr = 0.04 + 0.96 * (1 - vdh) ** 5
        spec = a2 * Fr / (4 * math.pi * dd * dd * (ndl * (1 - kk) + kk) * (ndv * (1 - kk) + kk))
        spec = torch.where((ndl > 0) & (ndv > 0), spec, torch.zeros_like(spec))
        rgb = (alb / math.pi + spec[:, None]) * rgb_l * ndl[:, None] + sc.ambient * alb
    out, ouv = torch.zeros((H * W, 3), **f8), torch.zeros((H * W, 2), **f8)
    out[pix], ouv[pix] = rgb, uv
    return out.reshape(H, W, 3), ouv.reshape(H, W, 2)


def exact(case, seed):
    """Rendered colours and UVs in 64 bits.  Estimates are whole numbers (fixed-point sums over random signs),
    and what is decoded or stepped from them has no value without them: None in their place."""
    if case["layers"] or case["subdiv"]:
        return None
    if case["kind"] == "render":
        sc = _scene(case, seed)
        got = [_render64(sc, v) for v in sc.views]
        return [[rgb, None, uv] for rgb, uv in got]
    if case["kind"] == "autograd":
        sc = _scene(case, seed)
        if case["form"] == "image":
            return [torch.stack([_render64(sc, v)[0] for v in sc.views]), None]
        tg = _scene(case, seed)
        tg.pos, tg.tex = sc.target_pos, sc.target_tex
        return [sum(((_render64(sc, v)[0] - _render64(tg, v)[0]) ** 2).sum() for v in sc.views), None]
    return None
