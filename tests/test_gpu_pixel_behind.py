"""Per-pixel order with keys at and below zero: large, thin, steeply tilted
Gaussians near the camera, whose plane a ray meets behind it, are maximal at a
negative z* there.  Such contributions are ordered in the window like any
other: images and contributor counts against the reference's exact per-pixel
sort, and the exact pass (one wave per pixel) is not needed for them."""
import numpy as np
import pytest

from gpu_helpers import baked, check_render, gpu_render, oracle_render, pair_total
from paper_2410_17932_amd import api, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [8, 16])
@pytest.mark.parametrize("planes,copies", [(1, 1), (5, 1), (2, 2)])
def test_keys_behind_the_camera(planes, copies, tile):
    W, H, n = 72, 56, 120
    rng = np.random.default_rng(planes)
    sc = synth.small_scene(200 + planes, n_gauss=n, width=W, height=H, f=64.0, sh_degree=1,
                           n_views=2)
    g, views = sc["gaussians"], sc["views"]
    # sheets above the eye's axis, 1.2 x 1.2 wide and 0.02 thick, tilted a little
    k = planes * copies
    tilt = np.tile(rng.uniform(-0.1, 0.1, planes), copies)
    y, z = np.tile(rng.uniform(0.2, 0.4, planes), copies), np.tile(rng.uniform(0.6, 0.9, planes), copies)
    g["mean"][:, :k] = np.stack([0 * y, -y, z])
    g["logscale"][:, :k] = np.log([[1.2], [0.02], [1.2]])
    g["quat"][:, :k] = np.stack([np.cos(tilt / 2), np.sin(tilt / 2), 0 * tilt, 0 * tilt])
    g["logit"][:k] = -1.5
    raster = dict(sc["raster"], tile=tile, order=api.ORDER_PIXEL)
    cov, op = baked(g)
    D = synth.views_dims(views)
    o, rect, _ = oracle_render(g, cov, op, views, raster)
    total = pair_total(rect, D, tile)
    gpu, ws = gpu_render(g, cov, op, views, raster, max_pairs=total + 1000)
    assert int(ws.status.item()) == 0
    check_render(o, gpu)
    # the depth image is a mean of z*: it falls below zero where the sheets prevail
    assert (o["depth"] < 0).mean() > 0.05
    assert ws.exact_pass_count() <= 0.02 * 2 * W * H
