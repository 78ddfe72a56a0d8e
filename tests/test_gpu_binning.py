"""Tile lists of the periphery bit-exact against the CPU reference where the
binning's work units change shape: a partial round of 64 pairs, a unit one
pair over or under full, every pair on all 64 tiles of its super-tile (one
round fills the stage), and mixtures."""
import numpy as np
import pytest

import oracle
from paper_2410_17932_amd import synth

from gpu_helpers import baked, gpu_render, oracle_render, pair_total

pytestmark = pytest.mark.gpu


def _check(sc, g, tile):
    views, raster = sc["views"], dict(sc["raster"], tile=tile)
    cov, op = baked(g)
    _, rect, zb = oracle_render(g, cov, op, views, raster, pix=np.zeros((1, 3), np.int32))
    D = synth.views_dims(views)
    total = pair_total(rect, D, tile)
    _, ws = gpu_render(g, cov, op, views, raster, max_pairs=total + 64)
    assert int(ws.status.item()) == 0 and ws.pair_count() == total
    ranges, ids = ws.tile_lists()
    per = ws.layout.tiles_x * ws.layout.tiles_y
    sel = np.array([[v, t] for v in range(len(views)) for t in range(per)], np.int32)
    off, want = oracle.tile_lists(rect, zb, D, tile, sel)
    for s in range(len(sel)):
        b, e = ranges[s]
        assert np.array_equal(ids[b:e], want[off[s]:off[s + 1]]), f"tile list {s} differs"


# n, added to the log-scales (0: a few tiles each; 4: the whole image), tile
@pytest.mark.parametrize("n,grow,tile", [(1, 4.0, 8), (63, 4.0, 8), (65, 4.0, 8), (255, 4.0, 8),
                                         (257, 4.0, 8), (900, 1.2, 8), (1500, 0.0, 8),
                                         (700, 2.0, 16), (900, "mixed", 8), (3000, "mixed", 32)])
def test_tile_lists_over_unit_shapes(n, grow, tile):
    sc = synth.small_scene(n, n_gauss=n, width=200, height=136, f=150.0, n_views=2)
    g = dict(sc["gaussians"])
    add = np.random.default_rng(n).uniform(-1, 4, n) if grow == "mixed" else grow
    g["logscale"] = (g["logscale"] + add).astype(np.float32)
    _check(sc, g, tile)


# two views of n: around the rows of 1024 and the limits of the one-workgroup
# sort (8192 depth keys, 16384 pairs); every third Gaussian shares its depth
# key with others, so the lists also show the sort's stability
@pytest.mark.parametrize("n", [2, 511, 512, 513, 3000, 4096, 4097])
def test_tile_lists_over_sort_sizes(n):
    sc = synth.small_scene(n, n_gauss=n, width=200, height=136, f=150.0, n_views=2)
    g = dict(sc["gaussians"])
    mean = g["mean"].copy()
    mean[2, ::3] = 3.5
    g["mean"] = mean
    _check(sc, g, 16)
