"""Edges of the kernels' splits and dispatch rules (bin rectangles, shared
walks, remainders), bit for bit against the CPU oracle.  Every comparison is
exact: both sides evaluate the same fp32 operation sequence and integer sums."""
import numpy as np
import pytest
import torch

import oracle
from paper_2404_09758_amd import api, batch
from paper_2404_09758_amd import scenes as S

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
