"""Edges of the kernels' splits and dispatch rules (bin rectangles, shared
walks, remainders), bit for bit against the CPU oracle.  Every comparison is
exact: both sides evaluate the same fp32 operation sequence and integer sums."""
import numpy as np
import pytest
import torch

import oracle
from paper_2404_09758_amd import api, batch
from paper_2404_09758_amd import scenes as S
from tests import helpers as H

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def mixed_soup(n, sizes, views, seed=0, shading=S.SHADING_UNLIT, tex_shape=(24, 40, 3)):
    """n independent triangles of log-uniform size (as a share of the view),
    the first ones consecutive and large, seen through views of (W, H)."""
    rng = np.random.default_rng(900 + seed)
    half = S.CAM_DIST * np.tan(np.radians(S.FOVY_DEG) / 2)
    size = half * np.exp(rng.uniform(np.log(sizes[0]), np.log(sizes[1]), n))
    size[: min(n, 3)] = half * sizes[1]
    centre = np.stack([rng.uniform(-half, half, n), rng.uniform(-half, half, n), rng.uniform(-0.3, 0.3, n)], 1)
    offs = rng.normal(0.0, 1.0, (n, 3, 3)) * size[:, None, None]
    offs[:, :, 2] *= 0.05
    pos = (centre[:, None, :] + offs).reshape(-1, 3).astype(np.float32)
    tri = np.arange(3 * n, dtype=np.int32).reshape(n, 3)
    cuv = rng.uniform(-0.2, 1.2, (n, 3, 2)).astype(np.float32)
    tex = [rng.uniform(0.05, 0.95, tex_shape).astype(np.float32)]
    ttex = [rng.uniform(0.05, 0.95, tex_shape).astype(np.float32)]
    vs = [S.look_at_view(w, h, 5.0 * k, 3.0) for k, (w, h) in enumerate(views)]
    eps = [2e-3, 1.0 / 255.0]
    return S.Scene("mixed", tri, cuv, pos, tex, pos, ttex, vs, shading=shading, eps=eps, lr=list(eps), n_pairs=1)


# Binning: blocks of 256 triangles (255, 256, 257 and a last block of one),
# tiles per triangle below and above the bound of the per-thread walk, block
# rectangles of up to 4096 tiles (65 x 63 tiles of 8 px) and beyond (66 x 65).
@pytest.mark.parametrize("n,sizes,tile,cap", [
    (1, (0.5, 0.5), 8, 256), (255, (0.002, 0.02), 16, 256), (256, (0.002, 0.6), 16, 256), (257, (0.002, 0.6), 8, 256),
    (257, (0.01, 0.05), 32, 256), (513, (0.002, 0.02), 8, 2), (300, (0.3, 1.5), 8, 64)])
def test_binning_edges_bit_exact(n, sizes, tile, cap):
    print(f"[kernels] binning n {n} sizes {sizes} tile {tile} cap {cap}", flush=True)
    views = [(520, 504), (528, 520)]
    sc = mixed_soup(n, sizes, views, seed=n)
    o = oracle.Oracle(sc)
    tg = [o.render(sc.flat_params(True), v)[0] for v in sc.views]
    Qo, Ko, _, _ = o.estimate(sc.flat_params(), sc.views, tg, 7, 3, 1, sc.eps)
    dtg = torch.cat([torch.tensor(t, device=DEV).reshape(-1) for t in tg])
    th = torch.tensor(sc.flat_params(), device=DEV)
    for items in (0, 1):
        ctx = api.Context(sc, DEV, tuning=(tile, cap, items))
        Q, K = ctx.estimate_grad(th, sc.views, dtg, 7, 3, 1, sc.eps)
        assert np.array_equal(host(K).view(np.uint32), Ko)
        assert np.array_equal(host(Q), Qo)
    small = mixed_soup(40, (0.01, 0.4), [(90, 70)], seed=1)
    for scs in ([sc], [sc, small]):                  # the one-scene and the many-scene launch
        tgs = [dtg] + [torch.zeros(3 * 90 * 70, device=DEV)] * (len(scs) - 1)
        bt = batch.Batch(scs, 1, DEV, tile_px=tile, seed=7, first_step=3, bin_capacities=[cap] * len(scs), targets=tgs)
        for _ in range(2):                           # the second finds the bins as the first left them
            bt.Q[0].zero_()
            bt.K[0].zero_()
            bt.estimate()
            assert np.array_equal(host(bt.K[0]).view(np.uint32), Ko)
            assert np.array_equal(host(bt.Q[0]), Qo)


def raster_edges_scene(w, h, layers=0, seed=0):
    """Triangles given in pixels under the identity projection: spans of
    31999, 32000 and 32001 subpixels (the bound of the 32-bit edge functions),
    boxes of 1 to 20 pixels that end at and one pixel either side of tile
    edges and of the view's right edge, and a large one behind them all."""
    rng = np.random.default_rng(70 + seed)
    px = []
    for span in (31999, 32000, 32001):
        s = span / 256.0
        x, y = rng.uniform(-20, w - 60), rng.uniform(-20, h - 60)
        px.append([(x, y), (x + s, y + 0.3 * s), (x + 0.4 * s, y + s)])
        px.append([(x, y + s), (x + s, y), (x + s - 3.0, y + 4.0)])          # a long thin one
    for width in range(1, 21):
        for edge in (32, 64, w, w + 2):
            for d in (-1, 0, 1):
                x1, y0 = edge + d, rng.uniform(0, h)
                px.append([(x1 - width, y0), (x1, y0 + rng.uniform(-2, 9)), (x1 - width * rng.random(), y0 + width)])
    px.append([(-w, -h), (3 * w, -h), (-w, 3 * h)])
    px = np.asarray(px, np.float64)
    n = len(px)
    z = np.concatenate([rng.uniform(-0.8, 0.5, n - 1), [0.9]])
    pos = np.empty((n, 3, 3))
    pos[:, :, 0] = 2 * px[:, :, 0] / w - 1
    pos[:, :, 1] = 1 - 2 * px[:, :, 1] / h
    pos[:, :, 2] = z[:, None] + rng.uniform(-0.05, 0.05, (n, 3))
    c = 4 if layers else 3
    tex = [rng.uniform(0.05, 0.95, (20, 28, c)).astype(np.float32)]
    ttex = [rng.uniform(0.05, 0.95, (20, 28, c)).astype(np.float32)]
    tri = np.arange(3 * n, dtype=np.int32).reshape(n, 3)
    pos = pos.reshape(-1, 3).astype(np.float32)
    eps = [1.5 / w, 1.0 / 255.0]
    return S.Scene("edges", tri, rng.uniform(0, 1, (n, 3, 2)).astype(np.float32), pos, tex, pos, ttex,
                   [H.ndc_view(w, h)], shading=S.SHADING_UNLIT, eps=eps, lr=list(eps), n_pairs=1, layers=layers)


# Raster: slots that run past the tile's and the view's right edge, triangles
# at the bound of the staged raster, large ones mixed with small ones.
@pytest.mark.parametrize("tile,cap,layers", [(8, 256, 0), (16, 256, 0), (32, 256, 0), (16, 3, 0), (8, 256, 2),
                                             (16, 256, 3)])
def test_raster_edges_bit_exact(tile, cap, layers):
    print(f"[kernels] raster tile {tile} cap {cap} layers {layers}", flush=True)
    sc = raster_edges_scene(187, 153, layers)
    o = oracle.Oracle(sc)
    v = sc.views[0]
    ctx = api.Context(sc, DEV, tuning=(tile, cap, 0))
    th = torch.tensor(sc.flat_params(), device=DEV)
    rgb, ids, uv = ctx.render(th, v)
    ro, io, uo = o.render(sc.flat_params(), v)
    assert np.array_equal(host(ids).view(np.uint32), io)
    assert np.array_equal(host(rgb), ro) and np.array_equal(host(uv), uo)
    tg = [o.render(sc.flat_params(True), v)[0]]
    Qo, Ko, _, _ = o.estimate(sc.flat_params(), sc.views, tg, 11, 2, 2, sc.eps)
    Q, K = ctx.estimate_grad(th, sc.views, torch.tensor(tg[0], device=DEV).reshape(-1), 11, 2, 2, sc.eps)
    assert np.array_equal(host(K).view(np.uint32), Ko)
    assert np.array_equal(host(Q), Qo)


# Subdivision scatter: control lists shorter and longer than a row of 16 lanes
# (a fan's hub raises the valence), pairs with one side background, tiles whose
# every pixel is a pair of its own, and the three tile sizes' pair tables.
def fan_scene(n, levels, res, seed=0):
    """A closed double pyramid over an n-gon: two hub vertices of valence n."""
    rng = np.random.default_rng(40 + seed)
    ang = 2 * np.pi * np.arange(n) / n
    pos = np.concatenate([np.stack([np.cos(ang), 0.25 * np.sin(3 * ang), np.sin(ang)], 1), [[0, 0.9, 0], [0, -0.9, 0]]])
    tri = [(i, n, (i + 1) % n) for i in range(n)] + [((i + 1) % n, n + 1, i) for i in range(n)]
    tri = np.array(tri, np.int32)
    cuv = rng.uniform(0, 1, (len(tri), 3, 2)).astype(np.float32)
    tex = [rng.uniform(0.05, 0.95, (40, 24, 3)).astype(np.float32)]
    ttex = [rng.uniform(0.05, 0.95, (40, 24, 3)).astype(np.float32)]
    pos = pos.astype(np.float32)
    tpos = (pos + rng.normal(0, 0.03, pos.shape)).astype(np.float32)
    eps = [0.03, 1.0 / 255.0]
    return S.Scene("fan", tri, cuv, pos, tex, tpos, ttex, [S.look_at_view(res, res - 13, 20.0, 35.0)],
                   shading=S.SHADING_LAMBERT, eps=eps, lr=list(eps), n_pairs=1, subdiv_levels=levels)


@pytest.mark.parametrize("n,levels,res,tile", [(3, 1, 40, 8), (24, 1, 90, 16), (24, 2, 60, 32), (40, 2, 100, 16),
                                               (40, 2, 33, 8)])
def test_subdivision_scatter_bit_exact(n, levels, res, tile):
    print(f"[kernels] subdivision n {n} levels {levels} res {res} tile {tile}", flush=True)
    sc = fan_scene(n, levels, res)
    o = oracle.Oracle(sc)
    tg = [o.render(sc.flat_params(True), v)[0] for v in sc.views]
    Qo, Ko, _, _ = o.estimate(sc.flat_params(), sc.views, tg, 3, 1, 2, sc.eps)
    ctx = api.Context(sc, DEV, tuning=(tile, 256, 0))
    Q, K = ctx.estimate_grad(torch.tensor(sc.flat_params(), device=DEV), sc.views,
                             torch.tensor(tg[0], device=DEV).reshape(-1), 3, 1, 2, sc.eps)
    assert np.array_equal(host(K).view(np.uint32), Ko)
    assert np.array_equal(host(Q), Qo)
    assert np.count_nonzero(Qo) > 0


# Sign bytes: groups at and around a block's chunk (8192), texel classes of
# their own, four-channel albedo; the texel box: rectangles at its limit, the
# UV seam, clamped rows, a texture finer than the pixels (hashed instead).
@pytest.mark.parametrize("tex_shapes,shading,layers,tile,freq", [
    (((8192, 1, 3),), 1, 0, 16, 6), (((91, 90, 3),), 1, 0, 8, 6), (((1, 8193, 3),), 0, 0, 16, 6),
    (((96, 128, 3), (64, 50, 3), (200, 3, 1)), 2, 0, 16, 5), (((128, 128, 3), (128, 128, 3), (32, 32, 1)), 2, 0, 32, 5),
    (((33, 47, 4),), 1, 3, 16, 5), (((600, 700, 4),), 0, 2, 8, 4), (((1024, 900, 3),), 1, 0, 16, 8),
    (((2, 2, 3),), 1, 0, 16, 6)])
def test_signs_and_texel_box_bit_exact(tex_shapes, shading, layers, tile, freq):
    print(f"[kernels] textures {tex_shapes} shading {shading} layers {layers} tile {tile}", flush=True)
    sc = H.sphere_scene(freq, 0, res=(91, 75), shading=shading, tex_shapes=tex_shapes, seed=8, views=2)
    sc.layers = layers
    o = oracle.Oracle(sc)
    tg = [o.render(sc.flat_params(True), v)[0] for v in sc.views]
    Qo, Ko, _, _ = o.estimate(sc.flat_params(), sc.views, tg, 21, 4, 2, sc.eps)
    ctx = api.Context(sc, DEV, tuning=(tile, 256, 0))
    th = torch.tensor(sc.flat_params(), device=DEV)
    dtg = torch.cat([torch.tensor(t, device=DEV).reshape(-1) for t in tg])
    Q, K = ctx.estimate_grad(th, sc.views, dtg, 21, 4, 2, sc.eps)
    assert np.array_equal(host(K).view(np.uint32), Ko)
    assert np.array_equal(host(Q), Qo)


# Plain launches share a setup of as many items as fit its scratch: 5 views x
# 7 pairs in launches of 1, 2, 3 and 4 items, with bins large enough that the
# items need several setups.
@pytest.mark.parametrize("items,cap", [(1, 256), (2, 65536), (3, 16384), (4, 65536)])
def test_plain_launches_share_setups_bit_exact(items, cap):
    print(f"[kernels] items {items} cap {cap}", flush=True)
    sc = H.sphere_scene(6, 0, res=(120, 104), shading=2, tex_shapes=((32, 32, 3), (32, 32, 3), (16, 16, 1)), seed=5,
                        views=5)
    o = oracle.Oracle(sc)
    tg = [o.render(sc.flat_params(True), v)[0] for v in sc.views]
    Qo, Ko, _, _ = o.estimate(sc.flat_params(), sc.views, tg, 2, 6, 7, sc.eps)
    ctx = api.Context(sc, DEV, tuning=(16, cap, items))
    th = torch.tensor(sc.flat_params(), device=DEV)
    dtg = torch.cat([torch.tensor(t, device=DEV).reshape(-1) for t in tg])
    Q, K = ctx.estimate_grad(th, sc.views, dtg, 2, 6, 7, sc.eps)
    assert np.array_equal(host(K).view(np.uint32), Ko)
    assert np.array_equal(host(Q), Qo)


# Launches that fill the chip sum their pixels by pairs of triangles first: 9
# items of 256 px hold more tiles than that takes at each tile size.  The soup's
# triangles share no vertices, the sphere's share most.
@pytest.mark.parametrize("mesh", ["sphere", "soup"])
@pytest.mark.parametrize("tile", [8, 16, 32])
def test_vertices_by_pairs_bit_exact(mesh, tile):
    print(f"[kernels] by pairs {mesh} tile {tile}", flush=True)
    if mesh == "soup":
        sc, pairs = S.make_soup(700, res=256, seed=4, pairs=9), 9
        tg = [sc.target_image]
        o = oracle.Oracle(sc)
    else:
        sc, pairs = H.sphere_scene(12, 0, res=(256, 250), shading=1, tex_shapes=((64, 64, 3),), seed=4, views=3), 3
        o = oracle.Oracle(sc)
        tg = [o.render(sc.flat_params(True), v)[0] for v in sc.views]
    Qo, Ko, _, _ = o.estimate(sc.flat_params(), sc.views, tg, 8, 2, pairs, sc.eps)
    ctx = api.Context(sc, DEV, tuning=(tile, 256, 0))
    dtg = torch.cat([torch.as_tensor(t, device=DEV).reshape(-1) for t in tg])
    Q, K = ctx.estimate_grad(torch.tensor(sc.flat_params(), device=DEV), sc.views, dtg, 8, 2, pairs, sc.eps)
    assert np.array_equal(host(K).view(np.uint32), Ko)
    assert np.array_equal(host(Q), Qo)


# The deep kernels for up to two and up to four layers, at each number of layers.
@pytest.mark.parametrize("layers", [1, 2, 3, 4])
@pytest.mark.parametrize("tile,shading", [(8, 0), (16, 1), (16, 0)])
def test_layer_counts_bit_exact(layers, tile, shading):
    print(f"[kernels] layers {layers} tile {tile} shading {shading}", flush=True)
    sc = H.sphere_scene(9, 0, res=(83, 69), shading=shading, tex_shapes=((40, 56, 4),), seed=11, views=2)
    sc.layers = layers
    o = oracle.Oracle(sc)
    tg = [o.render(sc.flat_params(True), v)[0] for v in sc.views]
    Qo, Ko, _, _ = o.estimate(sc.flat_params(), sc.views, tg, 5, 3, 2, sc.eps)
    ctx = api.Context(sc, DEV, tuning=(tile, 256, 0))
    th = torch.tensor(sc.flat_params(), device=DEV)
    for v, t in zip(sc.views, tg):
        img = ctx.render(torch.tensor(sc.flat_params(True), device=DEV), v, ids=False, uv=False)[0]
        assert np.array_equal(host(img).reshape(-1), np.asarray(t).reshape(-1))
    dtg = torch.cat([torch.tensor(t, device=DEV).reshape(-1) for t in tg])
    Q, K = ctx.estimate_grad(th, sc.views, dtg, 5, 3, 2, sc.eps)
    assert np.array_equal(host(K).view(np.uint32), Ko)
    assert np.array_equal(host(Q), Qo)


# Decode, step, fold and full-image sums work on a group's parameters as vectors
# of 3, 1 or 4: buffers that start off a 16-byte boundary, groups without a
# contribution, gradients past the type's range, and blocks with a zero eps.
@pytest.mark.parametrize("shapes,shading,layers,zero", [
    (((9, 7, 3), (9, 7, 3), (5, 3, 1)), 2, 0, 1), (((9, 7, 3), (9, 7, 3), (9, 7, 1)), 2, 0, -1),
    (((11, 5, 4),), 1, 2, -1), (((11, 5, 3),), 0, 0, 0)])
@pytest.mark.parametrize("kind,averaging", [(api.ADAM, api.AVG_COUNT), (api.SGD, 1 - api.AVG_COUNT)])
def test_parameter_vectors_bit_exact(shapes, shading, layers, zero, kind, averaging):
    sc = H.sphere_scene(3, 0, res=(24, 20), shading=shading, tex_shapes=shapes, seed=2, views=1)
    sc.layers = layers
    eps = list(sc.eps)
    if zero >= 0:
        eps[zero] = 0.0
    eps[-1] = 1e-38 if zero != len(eps) - 1 else 0.0      # (an infinite gradient for large sums)
    ctx, o = api.Context(sc, DEV), oracle.Oracle(sc)
    rng = np.random.default_rng(9)
    th, m, v = [rng.normal(size=ctx.d).astype(np.float32) for _ in range(3)]
    v = np.abs(v)
    Q = rng.integers(-2**45, 2**45, ctx.d) * rng.integers(0, 2, ctx.d)
    K = (rng.integers(0, 9, ctx.G) * rng.integers(0, 2, ctx.G)).astype(np.uint32)

    def off(a):                                           # the array one element into a buffer
        return torch.cat([torch.zeros(1, dtype=torch.as_tensor(a).dtype), torch.as_tensor(a)]).to(DEV)[1:]

    d_th, d_m, d_v, d_Q, d_K = off(th), off(m), off(v), off(Q), off(K.view(np.int32))
    g = ctx.decode_grad(d_Q, d_K, eps, averaging=averaging, n_pairs=3)
    assert np.array_equal(host(g), o.decode(Q, K, eps, averaging, 3), equal_nan=True)
    ctx.step(d_th, d_m, d_v, 2, d_Q, d_K, eps, 3, kind=kind, averaging=averaging, lr=sc.lr)
    o.step(th, m, v, 2, Q, K, eps, 3, kind=kind, averaging=averaging, lr=sc.lr)
    for a, b in ((d_th, th), (d_m, m), (d_v, v)):
        assert np.array_equal(host(a).view(np.uint32), b.view(np.uint32))
    assert not host(d_Q).any() and not host(d_K).any()


# Plain launches on several streams: calls that follow each other without a
# synchronisation, from the default and from another stream, with buffers made
# and dropped between them; and the same call recorded in a graph, which stays on
# one stream, replayed with eager calls in between.
@pytest.mark.parametrize("form", ["loss", "full"])
@pytest.mark.parametrize("items,views,pairs", [(1, 5, 6), (1, 2, 3), (2, 4, 7)])
def test_plain_launches_on_several_streams_bit_exact(form, items, views, pairs):
    print(f"[kernels] streams {form} items {items} views {views} pairs {pairs}", flush=True)
    sc = H.sphere_scene(8, 0, res=(400, 360), shading=1, tex_shapes=((48, 64, 3),), seed=6, views=views)
    ctx = api.Context(sc, DEV, tuning=(16, 256, items))
    one = api.Context(sc, DEV, tuning=(16, 256, 0))
    th = torch.tensor(sc.flat_params(), device=DEV)
    tg = torch.rand(sum(3 * v.width * v.height for v in sc.views), device=DEV)

    def call(c, t):
        return c.estimate_grad(th, sc.views, tg, 3, t, pairs, sc.eps, full_image=form == "full")

    want = [tuple(host(a) for a in call(one, t)) for t in range(4)]
    got = []
    for t in range(4):
        got.append(call(ctx, t))
        torch.empty(1 << 20, device=DEV).fill_(float("nan"))
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        for t in range(4):
            got.append(call(ctx, t))
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    for k, g in enumerate(got):
        assert all(np.array_equal(host(a), b) for a, b in zip(g, want[k % 4]))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        held = call(ctx, 2)
    for t in range(3):
        graph.replay()
        assert all(np.array_equal(host(a), b) for a, b in zip(held, want[2]))
        assert all(np.array_equal(host(a), b) for a, b in zip(call(ctx, t), want[t]))


# The loss's own launch shape: a 32-pixel tile is summed by 256 threads.
@pytest.mark.parametrize("tile,layers", [(8, 0), (16, 0), (32, 0), (8, 2), (16, 3)])
def test_loss_at_every_tile_size(tile, layers):
    print(f"[kernels] loss tile {tile} layers {layers}", flush=True)
    sc = H.sphere_scene(5, 0, res=(83, 69), shading=1, tex_shapes=((24, 20, 4 if layers else 3),), seed=3, views=2)
    sc.layers = layers
    o = oracle.Oracle(sc)
    tg = [o.render(sc.flat_params(True), v)[0] for v in sc.views]
    want = np.array([o.pixel_loss(sc.flat_params(), v, t).astype(np.float64).sum() for v, t in zip(sc.views, tg)])
    ctx = api.Context(sc, DEV, tuning=(tile, 256, 0))
    dtg = torch.cat([torch.tensor(t, device=DEV).reshape(-1) for t in tg])
    got = host(ctx.loss(torch.tensor(sc.flat_params(), device=DEV), sc.views, dtg))
    # the same terms in another order of summing: both sums within n u of the exact one
    n = 83 * 69
    assert np.all(np.abs(got - want) <= 2 * n * 2.0 ** -53 * np.abs(want))


# Every form of the tile kernel at every tile size and shading.
@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("shading", [0, 1, 2])
def test_forms_at_every_tile_size_bit_exact(tile, shading):
    print(f"[kernels] forms tile {tile} shading {shading}", flush=True)
    shapes = ((24, 20, 3), (24, 20, 3), (9, 11, 1))[: 3 if shading == 2 else 1]
    sc = H.sphere_scene(5, 0, res=(83, 69), shading=shading, tex_shapes=shapes, seed=3, views=2)
    o, ctx = oracle.Oracle(sc), api.Context(sc, DEV, tuning=(tile, 256, 0))
    tg = []
    for v in sc.views:
        rgb, ids, uv = ctx.render(torch.tensor(sc.flat_params(True), device=DEV), v)
        want = o.render(sc.flat_params(True), v)
        tg.append(want[0])
        for a, b in zip((rgb, ids, uv), want):
            assert np.array_equal(host(a).reshape(-1).view(np.uint32), np.asarray(b).reshape(-1).view(np.uint32))
    th = torch.tensor(sc.flat_params(), device=DEV)
    dtg = torch.cat([torch.tensor(t, device=DEV).reshape(-1) for t in tg])
    for kw in ({}, {"full_image": True}, {"image_grad": True}):
        Qo, Ko, _, _ = o.estimate(sc.flat_params(), sc.views, tg, 5, 3, 2, sc.eps, **kw)
        Q, K = ctx.estimate_grad(th, sc.views, dtg, 5, 3, 2, sc.eps, **kw)
        assert np.array_equal(host(K).view(np.uint32), Ko), kw
        assert np.array_equal(host(Q), Qo), kw


# A batch of mixed shadings takes the general kernels, as does a texture of more
# than 2^24 texels.
@pytest.mark.parametrize("tile", [8, 16, 32])
def test_batch_of_mixed_shadings_bit_exact(tile):
    scs = [H.sphere_scene(5, 0, res=(60, 50), shading=s, seed=s, views=2,
                          tex_shapes=((24, 20, 3), (24, 20, 3), (9, 11, 1))[: 3 if s == 2 else 1]) for s in (0, 1, 2)]
    tg = [[oracle.Oracle(sc).render(sc.flat_params(True), v)[0] for v in sc.views] for sc in scs]
    bt = batch.Batch(scs, 2, DEV, tile_px=tile, seed=9, first_step=1,
                     targets=[[torch.tensor(t, device=DEV) for t in ts] for ts in tg])
    bt.estimate()
    for b, sc in enumerate(scs):
        Qo, Ko, _, _ = oracle.Oracle(sc).estimate(sc.flat_params(), sc.views, tg[b], 9, 1, 2, sc.eps, scene_index=b)
        assert np.array_equal(host(bt.K[b]).view(np.uint32), Ko), b
        assert np.array_equal(host(bt.Q[b]), Qo), b


@pytest.mark.parametrize("tile", [8, 16, 32])
def test_texture_past_24_bit_offsets_bit_exact(tile):
    print(f"[kernels] large texture tile {tile}", flush=True)
    sc = H.sphere_scene(4, 0, res=(48, 40), shading=1, tex_shapes=((4100, 4099, 3),), seed=3, views=1)
    o, ctx = oracle.Oracle(sc), api.Context(sc, DEV, tuning=(tile, 256, 0))
    tg = [o.render(sc.flat_params(True), sc.views[0])[0]]
    Qo, Ko, _, _ = o.estimate(sc.flat_params(), sc.views, tg, 5, 3, 1, sc.eps)
    Q, K = ctx.estimate_grad(torch.tensor(sc.flat_params(), device=DEV), sc.views,
                             torch.tensor(tg[0], device=DEV).reshape(-1), 5, 3, 1, sc.eps)
    assert np.array_equal(host(K).view(np.uint32), Ko)
    assert np.array_equal(host(Q), Qo)


# A captured estimate whose bins overflow: replays between eager calls that raise
# the capacity and need larger scratch go on using what the graph was made with.
@pytest.mark.parametrize("form", ["loss", "full"])
@pytest.mark.parametrize("items", [0, 1])
def test_captured_estimate_outlives_new_scratch(form, items):
    print(f"[kernels] capture {form} items {items}", flush=True)
    sc = H.sphere_scene(8, 0, res=(150, 130), shading=2, tex_shapes=((32, 48, 3), (32, 48, 3), (16, 16, 1)), seed=6,
                        views=2)
    ctx = api.Context(sc, DEV, tuning=(16, 4, items))
    ref = api.Context(sc, DEV, tuning=(16, 256, 0))
    th = torch.tensor(sc.flat_params(), device=DEV)
    tg = torch.rand(sum(3 * v.width * v.height for v in sc.views), device=DEV)

    def call(c, t, pairs=3):
        return c.estimate_grad(th, sc.views, tg, 3, t, pairs, sc.eps, full_image=form == "full")

    def same(got, want):
        return all(np.array_equal(host(a), b) for a, b in zip(got, want))

    want = {(t, p): tuple(host(a) for a in call(ref, t, p)) for t in range(3) for p in (3, 40)}
    assert same(call(ctx, 0), want[0, 3])
    graphs = []
    for t in (1, 2):                                     # at the first capacity and at the raised one
        graph = torch.cuda.CUDAGraph()
        capacity = ctx.get_tuning()[1]
        with torch.cuda.graph(graph):
            out = call(ctx, t)
        assert ctx.get_tuning()[1] == capacity
        graphs.append((graph, out, want[t, 3]))
        for pairs in (3, 3, 40):
            assert same(call(ctx, 0, pairs), want[0, pairs])
            torch.empty(1 << 22, device=DEV).fill_(float("nan"))
            for g, o, w in graphs:
                g.replay()
                assert same(o, w)
    assert ctx.get_tuning()[1] > 4


# Full-image sums of 32-pixel tiles: a thread per pixel up to 512 blocks, four
# pixels a thread above; views that end within a tile.
@pytest.mark.parametrize("res,pairs", [((512, 512), 2), ((513, 512), 2), ((505, 250), 4), ((505, 250), 5), ((40, 30), 1)])
def test_full_image_of_large_tiles_bit_exact(res, pairs):
    print(f"[kernels] full image {res} pairs {pairs}", flush=True)
    sc = H.sphere_scene(7, 0, res=res, shading=2, tex_shapes=((40, 56, 3), (40, 56, 3), (9, 11, 1)), seed=12, views=1)
    o = oracle.Oracle(sc)
    tg = [o.render(sc.flat_params(True), sc.views[0])[0]]
    Qo, Ko, _, _ = o.estimate(sc.flat_params(), sc.views, tg, 5, 3, pairs, sc.eps, full_image=True)
    th = torch.tensor(sc.flat_params(), device=DEV)
    dtg = torch.tensor(tg[0], device=DEV).reshape(-1)
    for items in (0, 1):
        Q, K = api.Context(sc, DEV, tuning=(32, 256, items)).estimate_grad(th, sc.views, dtg, 5, 3, pairs, sc.eps,
                                                                           full_image=True)
        assert np.array_equal(host(K).view(np.uint32), Ko)
        assert np.array_equal(host(Q), Qo)


# Bins whose render's spill list is full look through the whole render: looks that
# are all hits (neighbouring triangles in one tile), batches that end when one
# finds no room, the remainder of a render; and spill lists that just hold.
@pytest.mark.parametrize("tile,layers", [(8, 0), (16, 0), (32, 0), (8, 2), (16, 4)])
@pytest.mark.parametrize("freq,res,scans", [(24, (70, 61), True), (31, (40, 33), True), (13, (40, 33), False)])
def test_overflowing_bins_bit_exact(freq, res, scans, tile, layers):
    print(f"[kernels] overflow freq {freq} res {res} tile {tile} layers {layers}", flush=True)
    sc = H.sphere_scene(freq, 0, res=res, shading=1, tex_shapes=((24, 20, 4 if layers else 3),), seed=3, views=1)
    sc.layers = layers
    o, v = oracle.Oracle(sc), sc.views[0]
    ctx = api.Context(sc, DEV, tuning=(tile, 4, 0))
    ctx.set_adaptive_bins(False)
    rgb, ids, uv = ctx.render(torch.tensor(sc.flat_params(True), device=DEV), v)
    ro, io, uo = o.render(sc.flat_params(True), v)
    assert np.array_equal(host(ids).view(np.uint32), io)
    assert np.array_equal(host(rgb), ro) and np.array_equal(host(uv), uo)
    Qo, Ko, _, _ = o.estimate(sc.flat_params(), sc.views, [ro], 5, 3, 2, sc.eps)
    for _ in range(2):                                   # the second finds bins and lists as the first left them
        Q, K = ctx.estimate_grad(torch.tensor(sc.flat_params(), device=DEV), sc.views,
                                 torch.tensor(ro, device=DEV).reshape(-1), 5, 3, 2, sc.eps)
        assert np.array_equal(host(K).view(np.uint32), Ko)
        assert np.array_equal(host(Q), Qo)
    st = ctx.stats()
    assert st["tile_overflows"] > 0 and (st["full_scans"] > 0) == scans
