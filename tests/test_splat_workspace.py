"""The splat's workspace grows with points and fragments, not with the view:
the image of hiding depths (kept where many points are culled without a
numbering) takes the fragments' place until they are written."""
import pytest

from paper_2410_17932_amd import api, synth


def _size(n, views, crops, levels, frags):
    return api.lib().vrs_splat_workspace_size(n, len(views), api.make_views(views),
                                              api.make_crops(crops), len(crops), levels, frags)


@pytest.mark.parametrize("W,H,crops,frags", [(2016, 2240, 16, 2_000_000), (1024, 1024, 4, 1_000_000)])
def test_no_view_sized_part_beside_the_fragments(W, H, crops, frags):
    n = 5_000_000
    views = [synth.pinhole(W, H, 0.5 * W) for _ in range(2)]
    crops = [synth.crop_at(i % 2, W / 2, H / 2, 512, W, H) for i in range(crops)]
    pixels = 2 * W * H
    area = sum(c.size ** 2 for c in crops)
    most = pixels * pixels // (4 * 2 * area)   # points from which the image is kept
    assert 0 < most < n
    per_point = 2 * 16
    for a, b in ((most - 10, most + 10), (1, n)):
        grown = _size(b, views, crops, 4, frags) - _size(a, views, crops, 4, frags)
        assert grown <= (b - a) * per_point + 4096
    # fewer fragments than the image has room for: no more than the image
    small = _size(n, views, crops, 4, 1)
    assert small <= n * per_point + 4 * pixels + 13 * api.pyramid_pixels(crops, 4) + (1 << 20)
