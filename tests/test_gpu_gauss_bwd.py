"""Adjoint of the periphery blend over its tile sizes (images that end inside a
sub-tile, whole sub-tiles past the edge, many tiles),
with and without a depth gradient, over a background, with opacities at the
clamp, and with lists longer than a staged batch.  Reference: oracle/diff.py in
float64; tolerance 1e-3 per element on a floor of 1e-3 of the largest, as for
every float32 adjoint."""
import numpy as np
import pytest
import torch

from gpu_helpers import baked, dev, oracle_render, pair_total
from oracle import diff
from paper_2410_17932_amd import api, synth
from paper_2410_17932_amd.autograd import RenderGaussians

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,tile,n,depth_grad,opaque", [
    (75, 59, 8, 400, True, False),
    (75, 59, 16, 400, False, True),
    (90, 33, 32, 700, True, True),
    (40, 24, 16, 2500, False, False),      # lists of several batches
    (1031, 1040, 16, 400, True, True),
    (1031, 1040, 32, 400, False, False),
])
def test_blend_backward_forms(W, H, tile, n, depth_grad, opaque):
    rng = np.random.default_rng(W + tile)
    sc = synth.small_scene(60 + tile, n_gauss=n, width=W, height=H, f=0.9 * W, sh_degree=1)
    g, views = sc["gaussians"], sc["views"]
    raster = dict(sc["raster"], tile=tile, bg=(0.3, 0.1, 0.6))
    cov, op = baked(g)
    if opaque:
        op[::3] = 1.0            # reach the clamp of 0.99 near their centres
    large = W * H > 100000
    pix = np.array([(0, x, y) for y in range(H) for x in range(W)], np.int32)
    if large:
        pix = pix[rng.choice(len(pix), 3000, replace=False)]
    o, rect, _ = oracle_render(g, cov, op, views, raster, pix=pix)
    V, D = synth.views_array(views), synth.views_dims(views)
    ok = o["margin"].reshape(-1) >= 1e-4                 # unambiguous pixels only
    cr, cd = rng.normal(size=(len(pix), 3)) * ok[:, None], rng.normal(size=len(pix)) * ok * 0.1
    P = {k: torch.tensor(np.asarray(v), dtype=torch.float64, requires_grad=True)
         for k, v in dict(mean=g["mean"], cov=cov, op=op, sh=g["sh"]).items()}
    out = diff.render(P["mean"], P["cov"], P["op"], P["sh"], 1, V, D, pix, raster)
    loss = (out["rgb"] * torch.tensor(cr)).sum()
    if depth_grad:
        loss = loss + (out["depth"] * torch.tensor(cd)).sum()
    loss.backward()
    opts = api.make_opts(**raster)
    ws = api.RenderWorkspace(n, views, opts, pair_total(rect, D, tile) + 64)
    T = [dev(a).requires_grad_() for a in (g["mean"], cov, op, g["sh"])]
    rgb, depth, _ = RenderGaussians.apply(*T, 1, views, opts, ws)
    full = np.zeros((4, H, W), np.float32)
    full[:3, pix[:, 2], pix[:, 1]] = cr.T
    full[3, pix[:, 2], pix[:, 1]] = cd
    loss = (rgb[0] * dev(full[:3])).sum()
    if depth_grad:
        loss = loss + (depth[0] * dev(full[3])).sum()
    for (k, ref), got in zip(P.items(), torch.autograd.grad(loss, T)):
        ref, got = ref.grad.numpy(), got.cpu().numpy().astype(np.float64)
        err = np.abs(got - ref) / np.maximum(np.abs(ref), 1e-3 * np.abs(ref).max())
        assert err.max() <= 1e-3, (k, err.max())
