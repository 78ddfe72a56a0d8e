"""The regulariser over a crop of more than 2^32 elements (37840 x 37840 x 3),
beside a small one, placed by the host and by the device table: the mean is
that of two marked elements, and the gradients reach the first and the last
element of either crop alike."""
import pytest
import torch

from paper_2410_17932_amd import api, synth

pytestmark = pytest.mark.gpu

S = 37840


@pytest.fixture
def memory_back():
    yield
    torch.cuda.empty_cache()


@pytest.mark.parametrize("placed", [False, True])
def test_regulariser_past_32_bits(memory_back, placed):
    if torch.cuda.mem_get_info()[0] < 90 << 30:
        pytest.skip("takes 70 GB of device memory")
    crops = [synth.Crop(0, 3, 1, 16, 11.0, 9.0), synth.Crop(0, 1, 0, S, 1 + S / 2, S / 2)]
    W, H = S + 1, S
    place = torch.tensor([[3, 1, 0, 0], [1, 0, 0, 0]], dtype=torch.int32, device="cuda") if placed else None
    n0, n1 = 3 * 16 * 16, 3 * S * S
    n = n0 + n1
    F = torch.zeros(n, device="cuda")
    P = torch.zeros((1, 3, H, W), device="cuda")
    F[-1], F[n0] = 3.0e9, 1.5e9
    P[0, 2, H - 1, W - 1] = 1.0e9   # the last element of the large crop, and no other's
    P[0, 0, :, 0] = 7.0e9           # outside both crops
    r = api.regulariser(F, P, crops, place=place)
    want = (4.5e9 - 1.0e9) / n
    assert abs(float(r[0]) - want) <= 1e-6 * want and abs(float(r[1]) - want) <= 1e-6 * want
    dF, dP = torch.zeros_like(F), torch.zeros_like(P)
    api.regulariser_backward(tuple(P.shape), crops, r, d_fovea=dF, d_periphery=dP, place=place)
    g = torch.tensor(1.0 / n, dtype=torch.float32, device="cuda")
    for i in (0, n0 - 1, n0, n0 + S * S, n - 2, n - 1):
        assert float(dF[i]) == float(g), i
    assert bool((dF == g).all())
    for c, y, x in ((0, 0, 1), (2, H - 1, W - 1), (1, H // 2, W - 1), (2, H - 1, 1)):
        assert float(dP[0, c, y, x]) == -float(g), (c, y, x)
    assert float(dP[0, :, :, 0].abs().max()) == 0.0
    assert float(dP[0, 1, 5, 7]) == -2 * float(g)   # under both crops
