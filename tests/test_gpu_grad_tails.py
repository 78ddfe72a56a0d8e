"""Gradients of tensors that hold more than a call uses: spherical harmonics
above the active degree, planes and rows past the ones read, a foveal buffer
longer than its crops, or one with no crops at all.  What the kernels do not
write has gradient zero.  Every new tensor starts as NaN here, so an element
that nobody writes shows.  Where the kernels write, the gradients are those of
the same call accumulating into zeros: to the bit for the combination, and
within 1e-5 of the largest for the periphery (sums over atomics)."""
import numpy as np
import pytest
import torch

from gpu_helpers import baked, dev
from paper_2410_17932_amd import api, synth
from paper_2410_17932_amd.autograd import CompositeFrame, RenderGaussians

pytestmark = pytest.mark.gpu


@pytest.fixture
def poisoned(monkeypatch):
    monkeypatch.setattr(torch, "empty_like", lambda t, **kw: torch.full_like(t, float("nan"), **kw))


@pytest.mark.parametrize("deg,rows,more", [(0, 16, 0), (1, 16, 0), (2, 9, 5), (3, 17, 1)])
def test_periphery_gradient_past_what_is_read(poisoned, deg, rows, more):
    """rows of sh coefficients, and `more` extra rows of every other input."""
    n = 257
    sc = synth.small_scene(deg, n_gauss=n, width=100, height=72, f=90.0, sh_degree=deg)
    g, views = sc["gaussians"], sc["views"]
    cov, op = baked(g)
    rng = np.random.default_rng(rows)
    pad = lambda a, r: np.concatenate([a, rng.normal(size=(r,) + a.shape[1:])]).astype(np.float32)
    sh = pad(g["sh"].reshape(-1, 3, n), rows - (deg + 1) ** 2)
    t = [dev(a).requires_grad_() for a in (pad(g["mean"], more), pad(cov, more), pad(op, more), sh)]
    opts = api.make_opts(**sc["raster"])
    ws = api.RenderWorkspace(n, views, opts, 100000)
    rgb, _, tf = RenderGaussians.apply(*t, deg, views, opts, ws)
    d_rgb = dev(rng.normal(size=tuple(rgb.shape)), torch.float32)
    got = torch.autograd.grad(rgb, t, d_rgb)
    want = [torch.zeros(x.shape, device=x.device) for x in t]
    api.render_gaussians_backward(*[x.detach() for x in t], deg, views, opts, ws, tf, d_rgb, None,
                                  *want)
    for a, b in zip(want, got):
        assert float((a - b).abs().max()) <= 1e-5 * float(a.abs().max())
        assert torch.equal(a == 0, b == 0)


@pytest.mark.parametrize("mode", [api.BLEND_LINEAR, api.BLEND_PAPER])
@pytest.mark.parametrize("n_crops,more", [(2, 7), (1, 5000), (0, 10), (2, 0)])
def test_combination_gradient_past_the_crops(poisoned, mode, n_crops, more):
    W, H = 64, 50
    rng = np.random.default_rng(more)
    crops = [synth.crop_at(0, 20.0, 25.0, 24, W, H), synth.crop_at(1, 30.0, 20.0, 40, W, H)][:n_crops]
    P = dev(rng.uniform(size=(2, 3, H, W)), torch.float32).requires_grad_()
    F = dev(rng.uniform(size=api.fovea_elements(crops) + more), torch.float32).requires_grad_()
    d_out = dev(rng.normal(size=(2, 3, H, W)), torch.float32)
    out = CompositeFrame.apply(P, F, crops, mode, 8.0, 0.75, 0.2)
    got = torch.autograd.grad(out, (P, F), d_out)
    want = [torch.zeros(x.shape, device=x.device) for x in (P, F)]
    api.composite_frame_backward(P.detach(), F.detach(), crops, d_out, *want, mode, 8.0, 0.75, 0.2)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
