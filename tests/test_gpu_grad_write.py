"""Adjoints that write their gradients against the same adjoints accumulating
into zeros: every element written (outputs start as NaN), the values the same.
The combination's, D-SSIM's and L1's arithmetic is the same, so they agree to
the bit; the periphery's sums over atomics differ between any two runs by
roundings (2^-24 each) of sums of up to some thousand terms: 1e-5 of the
largest gradient."""
import numpy as np
import pytest
import torch

from gpu_helpers import baked, dev
from paper_2410_17932_amd import api, synth

pytestmark = pytest.mark.gpu


def _nan(t):
    return torch.full_like(t, float("nan"))


@pytest.mark.parametrize("deg,n,depth", [(0, 300, False), (1, 257, True), (2, 600, True),
                                         (3, 1000, False)])
def test_periphery_gradients_written(deg, n, depth):
    sc = synth.small_scene(n, n_gauss=n, width=100, height=72, f=90.0, sh_degree=deg, n_views=2)
    g, views = sc["gaussians"], sc["views"]
    mean = g["mean"].copy()
    mean[2, ::5] = -1.0   # behind every camera: no pixel takes them
    cov, op = baked(g)
    t = [dev(mean), dev(cov), dev(op), dev(g["sh"])]
    opts = api.make_opts(**sc["raster"])
    ws = api.RenderWorkspace(n, views, opts, 200000)
    out = api.render_gaussians(*t, deg, views, opts, ws)
    rng = np.random.default_rng(n)
    d_rgb = dev(rng.normal(size=tuple(out["rgb"].shape)), torch.float32)
    d_depth = dev(rng.normal(size=tuple(out["depth"].shape)), torch.float32) if depth else None
    zero, nan = [torch.zeros_like(x) for x in t], [_nan(x) for x in t]
    api.render_gaussians_backward(*t, deg, views, opts, ws, out["tfinal"], d_rgb, d_depth, *zero)
    api.render_gaussians_backward(*t, deg, views, opts, ws, out["tfinal"], d_rgb, d_depth, *nan,
                                  accumulate=False)
    for a, b in zip(zero, nan):
        assert float((a - b).abs().max()) <= 1e-5 * float(a.abs().max())
    assert float(nan[0][:, ::5].abs().max()) == 0.0


@pytest.mark.parametrize("W,mode,n_crops", [(64, api.BLEND_PAPER, 2), (61, api.BLEND_LINEAR, 2),
                                            (64, api.BLEND_LINEAR, 0)])
def test_combination_gradients_written(W, mode, n_crops):
    rng = np.random.default_rng(W)
    H = 50
    crops = [synth.crop_at(0, 20.0, 25.0, 24, W, H), synth.crop_at(1, 30.0, 20.0, 40, W, H)][:n_crops]
    P = dev(rng.uniform(size=(2, 3, H, W)), torch.float32)
    F = dev(rng.uniform(size=max(1, sum(3 * c.size ** 2 for c in crops))), torch.float32)
    g = dev(rng.normal(size=(2, 3, H, W)), torch.float32)
    zero, nan = (torch.zeros_like(P), torch.zeros_like(F)), (_nan(P), _nan(F))
    api.composite_frame_backward(P, F, crops, g, *zero, mode=mode)
    api.composite_frame_backward(P, F, crops, g, *nan, mode=mode, accumulate=False)
    assert torch.equal(zero[0], nan[0])
    if n_crops:
        assert torch.equal(zero[1], nan[1])


@pytest.mark.parametrize("n,shift", [(1, 0), (7, 0), (4096, 0), (100003, 1)])
def test_loss_gradients_written(n, shift):
    rng = np.random.default_rng(n)
    x, y = (dev(rng.uniform(size=n + shift), torch.float32)[shift:] for _ in range(2))
    y[::3] = x[::3]
    scale = torch.tensor([0.7], device="cuda")
    zero, nan = torch.zeros_like(x), _nan(x)
    api.l1_loss(x, y, d_pred=zero, scale=float(scale))
    api.l1_loss_backward(x, y, nan, d_loss=scale)
    assert torch.equal(zero, nan)
    W, H = 67, 31
    a, b = (dev(rng.uniform(size=(3, H, W)), torch.float32) for _ in range(2))
    ws = api.DssimWorkspace(3, W, H)
    zero = torch.zeros_like(a)
    api.dssim_backward(a, b, ws, zero, d_loss=scale)
    # the loss and the gradient from one pass's maps
    loss, maps = api.dssim_forward_maps(a, b, 3, W, H)
    assert torch.equal(loss, api.dssim(a, b, ws))
    nan = _nan(a)
    api.dssim_backward_maps(a, b, 3, W, H, maps, nan, d_loss=scale)
    assert torch.equal(zero, nan)
