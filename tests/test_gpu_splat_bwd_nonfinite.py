"""What lies behind a fully opaque fragment (alpha of 1 or more) has no part in
the splat's adjoint, also where it is not finite: infinite features behind it
leave the gradients in front as they are, and a pixel gradient that is not
finite does not reach the points behind.  Lists shorter and longer than the 16
fragments that are scanned at a time, the opaque one anywhere in them."""
import numpy as np
import pytest
import torch

from gpu_helpers import dev
from paper_2410_17932_amd import api, synth

pytestmark = pytest.mark.gpu

W, H, L = 64, 48, 3


def _lists(front, behind):
    """Points one behind the other, the four pixels around the axis each."""
    n = front + 1 + behind
    views = [synth.pinhole(W, H, 60.0)]
    crops = [synth.crop_at(0, 32.0, 24.0, 16, W, H)]
    z = np.linspace(2.0, 4.0, n)
    pos = np.stack([0 * z, 0 * z, z]).astype(np.float32)
    r = (0.004 * z).astype(np.float32)
    op = np.full(n, 0.4, np.float32)
    op[front] = 5.0
    rng = np.random.default_rng(n)
    feat = rng.uniform(-1, 1, (n, 4)).astype(np.float16)
    return views, crops, pos, r, op, feat, rng


def _gradients(views, crops, pos, r, op, feat, d_pyr):
    n = len(r)
    ws = api.SplatWorkspace(n, views, crops, L, 5 * n + 16)
    args = (dev(pos), dev(r), dev(feat.view(np.int16)), dev(op), views, crops, L)
    pyr = api.splat_points(*args, None, None, ws)
    keys, ids = ws.lists()
    assert len(keys) == 4 * n and np.array_equal(ids.reshape(4, n), np.tile(np.arange(n), (4, 1)))
    g = dict(d_feat=torch.zeros((n, 4), device="cuda"), d_pos=torch.zeros((3, n), device="cuda"),
             d_radius=torch.zeros(n, device="cuda"), d_opacity=torch.zeros(n, device="cuda"))
    d = torch.zeros_like(pyr)
    d[torch.from_numpy(np.unique(keys)).cuda()] = dev(d_pyr)
    api.splat_points_backward(*args, d, ws, **g)
    return {k: np.moveaxis(v.cpu().numpy(), -1 if k == "d_pos" else 0, 0) for k, v in g.items()}


@pytest.mark.parametrize("front,behind", [(0, 1), (1, 1), (3, 20), (14, 1), (15, 1), (16, 3),
                                          (20, 40)])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_behind_an_opaque_fragment(front, behind, bad):
    views, crops, pos, r, op, feat, rng = _lists(front, behind)
    d_pyr = rng.normal(size=(4, 4)).astype(np.float32)
    want = _gradients(views, crops, pos, r, op, feat, d_pyr)
    spoilt = feat.copy()
    spoilt[front + 1:] = bad
    got = _gradients(views, crops, pos, r, op, spoilt, d_pyr)
    for k in want:
        assert np.array_equal(got[k][:front], want[k][:front]), k
        assert not got[k][front + 1:].any() and not want[k][front + 1:].any(), k
    assert np.array_equal(got["d_feat"], want["d_feat"])
    assert not front or np.abs(want["d_feat"][:front]).max() > 0
    # a pixel's gradient
    d_pyr[2, 1] = bad
    got = _gradients(views, crops, pos, r, op, feat, d_pyr)
    for k in got:
        assert not got[k][front + 1:].any(), k
