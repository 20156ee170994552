"""Which of the library's calls the autograd binding makes, on a stand-in context without a GPU."""
from __future__ import annotations

import pytest

torch = pytest.importorskip("torch")


class _Ctx:
    """z = sum of theta, gradient 2 (so that the two calls can be told apart)."""

    def __init__(self):
        self.calls = []

    def smooth(self, m, theta, K):
        self.calls.append("smooth")
        return theta.sum(1)

    def grad(self, m, theta, K):
        self.calls.append("grad")
        return theta.sum(1), torch.full_like(theta, 2.0)


def test_gradient_is_computed_only_where_it_can_be_asked_for():
    from paper_1401_8060_amd.autograd import smooth_snr
    theta, K = torch.rand(3, 6), torch.ones(3, dtype=torch.int32)
    leaf = theta.clone().requires_grad_(True)
    c = _Ctx()
    want = theta.sum(1)
    assert torch.equal(smooth_snr(c, None, theta, K), want)
    with torch.no_grad():
        z = smooth_snr(c, None, leaf, K)
    assert torch.equal(z, want) and not z.requires_grad
    with torch.inference_mode():
        assert torch.equal(smooth_snr(c, None, leaf, K), want)
    assert c.calls == ["smooth"] * 3
    z = smooth_snr(c, None, leaf, K)
    z.backward(torch.tensor([1.0, 2.0, 3.0]))
    assert c.calls[3:] == ["grad"]
    assert torch.equal(leaf.grad, torch.tensor([[2.0], [4.0], [6.0]]).expand(3, 6))


def test_four_argument_apply():
    from paper_1401_8060_amd.autograd import SmoothSNR
    leaf, K = torch.rand(3, 6).requires_grad_(True), torch.ones(3, dtype=torch.int32)
    SmoothSNR.apply(leaf, K, _Ctx(), None).sum().backward()
    assert torch.equal(leaf.grad, torch.full((3, 6), 2.0))
