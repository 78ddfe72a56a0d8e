"""The splat's gradients are tensors of their own: none is a view of another's
memory, so that they can be changed in place (also with tensors that need a
gradient), detached, kept and saved one by one.  The library's calls are
replaced here: nothing of the values is looked at."""
import pytest
import torch

from paper_2410_17932_amd import api
from paper_2410_17932_amd.autograd import SplatPoints


class _Ws:
    generation = 0


@pytest.mark.parametrize("with_op", [False, True])
def test_splat_gradients_are_their_own(monkeypatch, with_op):
    n = 5
    monkeypatch.setattr(api, "splat_points", lambda *a, **k: torch.zeros((7, 4)))

    def backward(*a, d_feat, d_pos, d_radius, d_opacity):
        for i, t in enumerate((d_feat, d_pos, d_radius, d_opacity)):
            if t is not None:
                assert t.is_contiguous() and t.dtype == torch.float32 and not t.any()
                t += i + 1.0
    monkeypatch.setattr(api, "splat_points_backward", backward)
    leaves = [torch.rand(3, n), torch.rand(n), torch.rand(n, 4), torch.rand(n)]
    leaves = [t.requires_grad_() for t in (leaves if with_op else leaves[:3])]
    out = SplatPoints.apply(leaves[0], leaves[1], leaves[2], leaves[3] if with_op else None, [], [],
                            3, None, None, _Ws())
    grads = torch.autograd.grad(out.sum(), leaves)
    places = {g.untyped_storage().data_ptr() for g in grads}
    assert len(places) == len(grads)
    for g, t, want in zip(grads, leaves, (2.0, 3.0, 1.0, 4.0)):
        assert g.shape == t.shape and bool((g == want).all())
        assert g.untyped_storage().nbytes() == 4 * g.numel()
        w = torch.ones_like(g).requires_grad_()
        g.mul_(w)                 # raises for a view made where gradients are off
        assert g.requires_grad
        g.detach_()
