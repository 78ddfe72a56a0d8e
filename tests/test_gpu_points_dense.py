"""The splat where layer pixels hold many fragments (ranked in depth buckets
and composited by a wave or a workgroup per pixel): lists bit-exact and the
pyramid within 1e-4 of the reference (as for short lists), at the edges of
that kernel's cases -- lists of at most 64, of up to 4096, beyond, thousands of
equal depths -- with opacities and with a numbering of the stored points."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import dev
from paper_2410_17932_amd import api, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,depths,opacity,permuted", [
    (300, "spread", False, False),        # lists of a few to 64
    (12000, "spread", True, True),        # hundreds
    (150000, "spread", False, True),      # past 4096 at the coarse layers
    (150000, "clustered", False, False),  # two far outliers leave one bucket with all others
    (9000, "equal", False, True),         # every depth the same: the numbering decides
    (150000, "equal", True, True),        # and more of them than one bucket holds
    (900, "levels", True, True),          # a few distinct depths
])
def test_dense_lists(n, depths, opacity, permuted):
    rng = np.random.default_rng(n + len(depths))
    W, H, L = 100, 90, 3
    views = [synth.pinhole(W, H, 90.0)]
    crops = [synth.crop_at(0, 50.0, 45.0, 16, W, H), synth.crop_at(0, 47.0, 49.0, 20, W, H)]
    p = synth.points(rng, n, "lognormal", xy=(-0.6, 0.6))
    p["radius"] *= 6.0
    if depths == "clustered":
        p["pos"][2] = 4.0 + rng.uniform(0.0, 1e-5, n)
        p["pos"][2, :2] = (2.0, 900.0)
        p["pos"][:2, :2] = 0.0
    elif depths == "equal":
        p["pos"][2] = 3.0
    elif depths == "levels":
        p["pos"][2] = rng.choice([2.5, 3.0, 4.0], n)
    op = rng.uniform(0.2, 1.0, n).astype(np.float32) if opacity else None
    V, D = synth.views_array(views), synth.views_dims(views)
    ci, _ = synth.crops_array(crops)
    off, oids = oracle.point_lists(p["pos"], p["radius"], V, D, ci, L, None, None)
    pyr_o = oracle.splat_points(p["pos"], p["radius"], p["feat"], V, D, ci, L, None, None,
                                opacity=op)
    perm = rng.permutation(n) if permuted else np.arange(n)
    stored = lambda a: dev(np.ascontiguousarray(a[..., perm]))
    ws = api.SplatWorkspace(n, views, crops, L, len(oids) + 13 * len(pyr_o))
    pyr = api.splat_points(stored(p["pos"]), stored(p["radius"]),
                           dev(np.ascontiguousarray(p["feat"][perm]).view(np.int16)),
                           None if op is None else stored(op), views, crops, L, None, None, ws,
                           point_ids=dev(perm.astype(np.int32)) if permuted else None)
    torch.cuda.synchronize()
    assert int(ws.status.item()) == 0
    keys, ids = ws.lists()
    assert np.array_equal(np.bincount(keys, minlength=len(off) - 1), np.diff(off))
    assert np.array_equal(perm[ids], oids), "fragment order differs"
    assert np.diff(off).max() > {300: 8, 900: 16, 9000: 256, 12000: 256, 150000: 4096}[n]
    assert np.abs(pyr.cpu().numpy() - pyr_o).max() <= 1e-4
