"""Adjoint of the decoder at the edges of its kernels' tiles: every number of
16-channel tiles (1 to 5), widths that fill none of them, layers that are no
multiple of 8 or 16 pixels, overlapping crops, and a layer large enough for
the 16-row tiles.  Reference: oracle/diff.py in float64.

Tolerance: the longest sum over products, 9 taps of 128 pre-activations, is
1152 terms long and rounds by at most 1152 2^-24 = 7e-5 of its absolute sum in
float32, whatever its order: 1e-4 of each gradient's largest magnitude."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import dev
from oracle import diff
from paper_2410_17932_amd import api, synth
from paper_2410_17932_amd.autograd import DecodeFovea

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("widths,L,sizes", [
    ((5,), 1, (17, 9)),                # one level: one channel tile, periphery beside the pyramid
    ((16, 3), 2, (34, 16)),            # two tiles, the coarse level narrower than its padding
    ((33, 17), 2, (18, 50)),           # three tiles, neither width a multiple of 4
    ((20, 48, 1), 3, (36, 20)),        # four tiles
    ((64, 64), 2, (40, 22)),           # five tiles
    ((8, 8), 2, (528,)),               # 33 x 33 tiles of 16 rows
])
@pytest.mark.parametrize("with_weights", [True, False])
def test_decoder_backward_tiles(widths, L, sizes, with_weights):
    rng = np.random.default_rng(len(widths) * 100 + widths[0])
    packed = synth.pack_decoder(synth.decoder_weights(rng, widths, 4))
    packed = (packed + rng.normal(0, 0.05, packed.shape)).astype(np.float32)
    W = H = max(sizes) + 7
    views = [synth.pinhole(W, H, 100.0)]
    crops = [synth.crop_at(0, W / 2 + i, H / 2 - i, s, W, H) for i, s in enumerate(sizes)]
    ci, _ = synth.crops_array(crops)
    pyr = rng.normal(size=(oracle.pyramid_pixels(ci, L), 4)).astype(np.float32)
    per = rng.uniform(size=(1, 3, H, W)).astype(np.float32)
    P = {k: torch.tensor(v, dtype=torch.float64, requires_grad=True)
         for k, v in dict(pyr=pyr, per=per, w=packed).items()}
    out = diff.decode(P["pyr"], P["per"], ci, L, widths, *diff.unpack_decoder(P["w"], widths))
    cot = rng.normal(size=tuple(out.shape))
    (out * torch.tensor(cot)).sum().backward()
    d_out = dev(cot, torch.float32)
    ws = api.DecoderWorkspace(widths, crops, api.VRS_F32)
    got = dict(pyr=dev(pyr), per=dev(per), w=dev(packed))
    if with_weights:
        leaves = [got[k].requires_grad_() for k in ("pyr", "per", "w")]
        o2 = DecodeFovea.apply(*leaves, L, views, crops, ws)
        g = dict(zip(("pyr", "per", "w"), torch.autograd.grad(o2, leaves, d_out)))
    else:
        # the entry point without a weight gradient, onto gradients that hold something
        api.decode_fovea(got["pyr"], L, got["per"], views, crops, got["w"], ws)
        g = dict(pyr=torch.ones_like(got["pyr"]), per=torch.ones_like(got["per"]))
        api.decode_fovea_backward(got["pyr"], L, got["per"], views, crops, got["w"], ws, d_out,
                                  g["pyr"], g["per"], None)
        g = {k: v - 1.0 for k, v in g.items()}
    for k, v in g.items():
        ref = P[k].grad.numpy()
        err = np.abs(v.cpu().numpy() - ref).max() / np.abs(ref).max()
        assert err <= 1e-4, (k, err)
