"""Selection of a million points and more without the depth cull (larger
workgroups, depths computed again for the survivors): a partial last workgroup,
several crops in both views, survivors in screen order (dense lists) and not.
Lists bit-exact, pyramid within 1e-4 of the reference."""
import numpy as np
import pytest

import oracle
from gpu_helpers import dev
from paper_2410_17932_amd import api, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dense,permuted", [(True, False), (False, True)])
def test_wide_selection(dense, permuted):
    n, W, H, L = (1 << 20) + 77, 256, 200, 3
    rng = np.random.default_rng(7)
    views = [synth.pinhole(W, H, 150.0), synth.pinhole(W, H, 150.0, (0.1, 0.05, -0.1))]
    crops = [synth.crop_at(0, 100.0, 90.0, 32, W, H), synth.crop_at(1, 130.0, 100.0, 20, W, H),
             synth.crop_at(0, 110.0, 95.0, 24, W, H)]
    far = 1.0 if dense else 10.0
    p = synth.points(rng, n, "uniform", xy=(-far, far))
    V, D = synth.views_array(views), synth.views_dims(views)
    ci, _ = synth.crops_array(crops)
    off, oids = oracle.point_lists(p["pos"], p["radius"], V, D, ci, L, None, None)
    pyr_o = oracle.splat_points(p["pos"], p["radius"], p["feat"], V, D, ci, L, None, None)
    capacity = len(oids) + (0 if dense else 3)
    assert (capacity > 12 * len(pyr_o)) == dense and len(oids) > len(pyr_o)
    perm = rng.permutation(n) if permuted else np.arange(n)
    stored = lambda a: dev(np.ascontiguousarray(a[..., perm]))
    ws = api.SplatWorkspace(n, views, crops, L, capacity)
    pyr = api.splat_points(stored(p["pos"]), stored(p["radius"]),
                           dev(np.ascontiguousarray(p["feat"][perm]).view(np.int16)), None, views,
                           crops, L, None, None, ws,
                           point_ids=dev(perm.astype(np.int32)) if permuted else None)
    assert int(ws.status.item()) == 0
    keys, ids = ws.lists()
    assert np.array_equal(np.bincount(keys, minlength=len(off) - 1), np.diff(off))
    assert np.array_equal(perm[ids], oids)
    assert np.abs(pyr.cpu().numpy() - pyr_o).max() <= 1e-4
