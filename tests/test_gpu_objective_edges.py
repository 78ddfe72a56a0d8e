"""The objective's kernels (combination and tone-mapping adjoints, L1,
D-SSIM) at the edges of their tiles, strips and vector loads, against the FP64
reference.

Tolerances.  The combination's gradients are products and sums of a few dozen
single-precision terms (under 32 roundings of 2^-24, 2e-6, of the largest
term); the edge term divides by the Sobel magnitude and multiplies by the
slope of S2, both fixed by the same few roundings of grey values (differences
of values near 1 against magnitudes of 0.1 and more: another factor 30), so
6e-5 of the largest gradient bounds it and 1e-4 is asked.  D-SSIM's loss and
gradient are asked what the other tests of it ask (2e-6 and 1e-3 of the
largest), as are tone mapping's.  L1's differences and their sums in fours
round four times, and up to 512 workgroups' sums are added in single
precision, half an ulp (2^-25) of the loss each: 2^-16 of it; its gradient is
two roundings of scale / n.
"""
import numpy as np
import pytest
import torch

from oracle import diff, post
from paper_2410_17932_amd import api, synth
from paper_2410_17932_amd.autograd import CompositeFrame

from gpu_helpers import dev

pytestmark = pytest.mark.gpu


def _crop(v, x0, y0, s, gx=None, gy=None):
    return synth.Crop(v, x0, y0, s, x0 + s / 2 if gx is None else gx,
                      y0 + s / 2 if gy is None else gy)


# W, H, crops (view, x0, y0, size): single pixels, tile remainders, crops at
# the image's corners, three crops over one another, rows not a multiple of 4,
# a gaze off the crop's centre
COMPOSITES = [
    (8, 8, [_crop(0, 0, 0, 1), _crop(1, 7, 7, 1), _crop(0, 3, 2, 2)]),
    (48, 40, [_crop(0, 0, 0, 16), _crop(0, 31, 23, 17), _crop(1, 8, 5, 33, 20.0, 25.0)]),
    (61, 53, [_crop(0, 2, 3, 40), _crop(0, 9, 5, 32), _crop(0, 15, 12, 23), _crop(1, 0, 0, 53)]),
    (64, 44, [_crop(1, 1, 1, 15), _crop(0, 6, 2, 42), _crop(0, 20, 4, 40)]),
]


@pytest.mark.parametrize("mode,gamma", [(api.BLEND_LINEAR, 0.2), (api.BLEND_PAPER, 0.0),
                                        (api.BLEND_PAPER, 0.2)])
@pytest.mark.parametrize("case", range(len(COMPOSITES)))
def test_composite_adjoint_edges(case, mode, gamma):
    W, H, crops = COMPOSITES[case]
    rng = np.random.default_rng(100 + case)
    ci, cf = synth.crops_array(crops)
    f32 = lambda a: a.astype(np.float32).astype(np.float64)
    P0 = f32(rng.uniform(size=(2, 3, H, W)))
    F0 = f32(rng.uniform(size=sum(3 * c.size ** 2 for c in crops)))
    g0 = f32(rng.normal(size=P0.shape))
    ref = {k: torch.tensor(a, requires_grad=True) for k, a in (("P", P0), ("F", F0))}
    diff.composite(ref["P"], ref["F"], ci, cf, mode=mode, ring=5.0, gamma=gamma).backward(
        torch.tensor(g0))
    got = {k: dev(a, torch.float32).requires_grad_() for k, a in (("P", P0), ("F", F0))}
    CompositeFrame.apply(got["P"], got["F"], crops, mode, 5.0, 0.75, gamma).backward(
        dev(g0, torch.float32))
    for k in ref:
        want = ref[k].grad.numpy()
        err = np.abs(got[k].grad.cpu().numpy() - want).max()
        assert err <= 1e-4 * max(1.0, np.abs(want).max()), (k, err)


@pytest.mark.parametrize("planes,H,W", [(1, 1, 1), (2, 13, 115), (1, 12, 116), (1, 68, 117),
                                        (3, 135, 233), (40, 200, 130), (1, 4, 600)])
def test_dssim_strips(planes, H, W):
    rng = np.random.default_rng(W + H)
    x = rng.uniform(0, 1, (planes, H, W)).astype(np.float32)
    y = np.clip(x + rng.normal(0, 0.15, x.shape), 0, 1).astype(np.float32)
    x[:, H // 2:] *= 0.01   # a dark part
    ws = api.DssimWorkspace(planes, W, H)
    assert abs(api.dssim(dev(x), dev(y), ws).item() - post.dssim(x, y)) < 2e-6
    want = post.dssim_backward(x, y)
    dx = torch.zeros(x.shape, device="cuda")
    api.dssim_backward(dev(x), dev(y), ws, dx)
    assert np.abs(dx.cpu().numpy() - want).max() < 1e-3 * np.abs(want).max() + 1e-12


@pytest.mark.parametrize("W,H,n", [(1, 1, 2), (63, 5, 48), (30, 34, 49), (130, 129, 256),
                                   (900, 611, 32)])
def test_tonemap_adjoint_columns(W, H, n):
    rng = np.random.default_rng(n)
    views = [synth.pinhole(W, H, 150.0, (0.03 * i, 0, 0)) for i in range(3)]
    x = rng.uniform(-0.2, 1.4, (3, 3, H, W)).astype(np.float32)
    p = post.gamma_params(3, n)
    p[:, 0] = rng.uniform(-0.6, 0.6, 3)
    p[:, 4:7] = rng.uniform(-0.3, 0.3, (3, 3))
    p = p.astype(np.float32)
    g = rng.normal(0, 1, x.shape).astype(np.float32)
    principal = np.array([[v.cx, v.cy] for v in views], np.float64)
    d_img, d_par = post.tonemap_backward(x, p, principal, g)
    di, dp = torch.empty(x.shape, device="cuda"), torch.zeros(p.shape, device="cuda")
    api.tonemap_backward(dev(x), views, dev(p), dev(g), d_img=di, d_params=dp)
    assert np.abs(di.cpu().numpy() - d_img).max() < 1e-5 * max(1.0, np.abs(d_img).max())
    assert np.abs(dp.cpu().numpy() - d_par).max() < 2e-4 * np.abs(d_par).max()


@pytest.mark.parametrize("n,shift", [(1, 0), (3, 0), (4, 1), (1023, 0), (524288 + 5, 0),
                                     (700001, 3)])
def test_l1_lengths_and_alignment(n, shift):
    rng = np.random.default_rng(n)
    a, b = (rng.uniform(size=n + shift).astype(np.float32) for _ in range(2))
    b[shift::3] = a[shift::3]
    pa, pb, d = dev(a)[shift:], dev(b)[shift:], torch.zeros(n + shift, device="cuda")[shift:]
    loss = api.l1_loss(pa, pb, d_pred=d, scale=3.0).item()
    e = (a.astype(np.float64) - b)[shift:]
    want = np.abs(e).mean()
    assert abs(loss - want) <= want * 2.0 ** -16
    g = np.sign(e) * 3.0 / n
    assert np.abs(d.cpu().numpy() - g).max() <= 3.0 / n * 2.0 ** -22
