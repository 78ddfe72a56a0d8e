"""Host-side argument checks of the entry points that write their gradients
and of D-SSIM with its maps kept, as tests/test_abi_args.py does for the
others: what the accumulating entries refuse, these refuse too."""
import ctypes

import pytest
import torch

from paper_2410_17932_amd import api, synth

pytestmark = pytest.mark.skipif(torch.cuda.is_available(),
                                reason="host-side checks only; run without a GPU")

EINVAL, EUNSUP = api.VRS_EINVAL, api.VRS_EUNSUPPORTED
P = ctypes.c_void_p(0x1000)   # stand-in device address, never dereferenced
BIG = 1 << 40


def _views(n=2, W=64, H=48):
    return api.make_views([synth.pinhole(W, H, 60.0, (0.03 * i, 0, 0)) for i in range(n)])


def _crops(spec):
    return api.make_crops([synth.Crop(v, x, y, s, x + s / 2, y + s / 2) for v, x, y, s in spec])


def _render(**kw):
    a = dict(mean=P, cov=P, op=P, sh=P, deg=0, n=10, views=_views(), nv=2, opts=api.make_opts(),
             tf=P, drgb=P, ddep=None, dmean=P, dcov=P, dop=P, dsh=P, ws=P, ws_bytes=BIG, pairs=100)
    a.update(kw)
    opts = ctypes.byref(a["opts"]) if a["opts"] is not None else None
    return [f(a["mean"], a["cov"], a["op"], a["sh"], a["deg"], a["n"], a["views"], a["nv"], opts,
              a["tf"], a["drgb"], a["ddep"], a["dmean"], a["dcov"], a["dop"], a["dsh"], a["ws"],
              a["ws_bytes"], a["pairs"], None)
            for f in (api.lib().vrs_render_gaussians_backward,
                      api.lib().vrs_render_gaussians_backward_write)]


@pytest.mark.parametrize("bad", [
    dict(opts=None), dict(opts=api.make_opts(tile=7)), dict(opts=api.make_opts(radix_bits=5)),
    dict(deg=-1), dict(deg=4), dict(n=-1), dict(views=None), dict(nv=0), dict(nv=9), dict(mean=None),
    dict(cov=None), dict(op=None), dict(sh=None), dict(tf=None), dict(drgb=None), dict(dmean=None),
    dict(dcov=None), dict(dop=None), dict(dsh=None), dict(ws=None), dict(ws_bytes=8),
    dict(pairs=-1)])
def test_render_backward_write_rejects(bad):
    assert _render(**bad) == [EINVAL, EINVAL]


def test_render_backward_write_orders_and_empty():
    assert _render(opts=api.make_opts(tile=8, order=api.ORDER_PIXEL)) == [EUNSUP, EUNSUP]
    v = _views()
    v[1].width = 80
    assert _render(views=v) == [EINVAL, EINVAL]
    assert _render(n=0, mean=None, cov=None, op=None, sh=None) == [api.VRS_OK, api.VRS_OK]
    for code in _render():
        assert code not in (api.VRS_OK, EINVAL, EUNSUP)   # past every check (no device here)


def _composite(**kw):
    a = dict(P_=P, nv=2, W=64, H=48, F=P, crops=[(0, 0, 0, 32)], mode=api.BLEND_PAPER, ring=8.0,
             m=0.75, g=P, dP=P, dF=P)
    a.update(kw)
    c = a["crops"]
    return [f(a["P_"], a["nv"], a["W"], a["H"], a["F"], _crops(c), len(c), None, a["mode"],
              a["ring"], a["m"], 0.2, a["g"], a["dP"], a["dF"], None)
            for f in (api.lib().vrs_composite_frame_backward,
                      api.lib().vrs_composite_frame_backward_write)]


@pytest.mark.parametrize("bad", [
    dict(mode=2), dict(mode=api.BLEND_LINEAR, ring=0.0), dict(m=1.0), dict(nv=0), dict(nv=9),
    dict(W=0), dict(H=0), dict(crops=[(0, 0, 0, 1)] * 33), dict(crops=[(0, 40, 0, 32)]),
    dict(crops=[(2, 0, 0, 16)]), dict(crops=[(0, 0, 0, 49)]), dict(crops=[(0, 0, 0, 0)]),
    dict(P_=None), dict(F=None), dict(g=None)])
def test_composite_backward_write_rejects(bad):
    assert _composite(**bad) == [EINVAL, EINVAL]


def test_composite_backward_write_without_outputs():
    assert _composite(dP=None, dF=None) == [api.VRS_OK, api.VRS_OK]
    for code in _composite() + _composite(crops=[(0, i, i, 16) for i in range(9)]):
        assert code not in (api.VRS_OK, EINVAL)


@pytest.mark.parametrize("bad", [dict(n=0), dict(n=-4), dict(x=None), dict(y=None), dict(d=None)])
def test_l1_backward_rejects(bad):
    a = dict(x=P, y=P, n=10, d=P)
    a.update(bad)
    assert api.lib().vrs_l1_loss_backward(a["x"], a["y"], a["n"], None, a["d"], None) == EINVAL


def test_l1_backward_passes():
    for d_loss in (None, P):
        assert api.lib().vrs_l1_loss_backward(P, P, 10, d_loss, P, None) not in (api.VRS_OK, EINVAL)


@pytest.mark.parametrize("bad", [dict(planes=0), dict(w=0), dict(h=-3), dict(planes=65536),
                                 dict(x=None), dict(y=None), dict(out=None), dict(maps=None),
                                 dict(short=1)])
def test_dssim_maps_reject(bad):
    a = dict(x=P, y=P, planes=3, w=64, h=48, out=P, maps=P, short=0)
    a.update(bad)
    size = api.lib().vrs_dssim_maps_size(a["planes"], a["w"], a["h"])
    if not any(k in bad for k in ("planes", "w", "h")):
        assert size > api.lib().vrs_dssim_workspace_size(3, 64, 48)
    else:
        assert size == 0
    size = BIG if size == 0 else size - a["short"]
    assert api.lib().vrs_dssim_forward_maps(a["x"], a["y"], a["planes"], a["w"], a["h"], a["out"],
                                            a["maps"], size, None) == EINVAL
    assert api.lib().vrs_dssim_backward_maps(a["x"], a["y"], a["planes"], a["w"], a["h"],
                                             a["maps"], size, None, a["out"], None) == EINVAL


def test_dssim_maps_pass():
    size = api.lib().vrs_dssim_maps_size(3, 64, 48)
    assert api.lib().vrs_dssim_forward_maps(P, P, 3, 64, 48, P, P, size, None) not in (api.VRS_OK, EINVAL)
    assert api.lib().vrs_dssim_backward_maps(P, P, 3, 64, 48, P, size, None, P, None) not in (api.VRS_OK, EINVAL)
