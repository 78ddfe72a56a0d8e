"""Tile lists where the binning lays its entries out in LDS first (over 4096
work units, at least four entries per pair): rounds that reach all 64 tiles of
their super-tile (32 pairs fill the stage), units of one pair, one over full
and full ones, mixtures of large and small rectangles, images that end inside a
super-tile.  Every list bit-exact against the CPU reference."""
import numpy as np
import pytest

import oracle
from paper_2410_17932_amd import synth

from gpu_helpers import baked, gpu_render, oracle_render, pair_total, tile_counts

pytestmark = pytest.mark.gpu

TILE, UNIT = 8, 256


# n, added to the log-scales, width, height (8 views)
@pytest.mark.parametrize("n,grow,W,H", [(1, 7.0, 1084, 1980), (65, 7.0, 1084, 1980),
                                        (256, 7.0, 1084, 1980), (257, 7.0, 1084, 1020),
                                        (600, "mixed", 1084, 1020)])
def test_staged_tile_lists(n, grow, W, H):
    sc = synth.small_scene(n, n_gauss=n, width=W, height=H, f=500.0, n_views=8)
    g, views = dict(sc["gaussians"]), sc["views"]
    if grow == "mixed":
        add = np.where(np.arange(n) % 2 == 0, 7.0, np.random.default_rng(n).uniform(-1, 3, n))
    else:
        add = grow
    g["logscale"] = (g["logscale"] + add).astype(np.float32)
    raster = dict(sc["raster"], tile=TILE)
    cov, op = baked(g)
    _, rect, zb = oracle_render(g, cov, op, views, raster, pix=np.zeros((1, 3), np.int32))
    D = synth.views_dims(views)
    total = pair_total(rect, D, TILE)
    units = int((-(-tile_counts(rect, D, 8 * TILE) // UNIT)).sum())
    assert units > 4096
    staged = total >= 4 * UNIT * units
    assert staged == (n > 16)   # (one pair a unit: 64 entries, the direct form)
    _, ws = gpu_render(g, cov, op, views, raster, max_pairs=total + 64)
    assert int(ws.status.item()) == 0 and ws.pair_count() == total
    ranges, ids = ws.tile_lists()
    per = ws.layout.tiles_x * ws.layout.tiles_y
    sel = np.stack([np.repeat(np.arange(8), per), np.tile(np.arange(per), 8)], 1).astype(np.int32)
    off, want = oracle.tile_lists(rect, zb, D, TILE, sel)
    assert np.array_equal(ranges[:, 1] - ranges[:, 0], np.diff(off))
    for s in range(len(sel)):
        b, e = ranges[s]
        assert np.array_equal(ids[b:e], want[off[s]:off[s + 1]]), f"tile list {s} differs"
