"""The launch that prepares a call of inference (operand, norms, folded parameters): K x D around a whole number of its
workgroups, row lengths around its batches of loads, and the same labels as cat_assign."""
import pytest
import torch

from paper_2509_26277_amd import cat_apply, cat_assign

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("alpha", [0.6, 1.0, 0.0])
@pytest.mark.parametrize("N,D,K", [(1, 4, 1), (40, 32, 32), (40, 33, 31), (40, 41, 25), (70, 1000, 50), (130, 1024, 17),
                                   (20, 1028, 16), (200, 512, 128), (300, 384, 200), (70, 7, 64)])
def test_inference_against_doubles(N, D, K, alpha):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N + D * K)
    r = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    N = max(N, K)
    cent, g, b = r(K, D), r(K, D), r(K, D)
    x = (cent[torch.arange(N, device="cuda") % K] + 0.1 * r(N, D)).contiguous()
    out, a = cat_apply(x, cent, g, b, alpha=alpha)
    d = ((x.double()[:, None, :] - cent.double()[None]) ** 2).sum(2)
    assert torch.equal(a.long(), d.argmin(1))  # (well separated)
    assert torch.equal(a, cat_assign(x, cent)[0])
    ge, be = 1 + alpha * (g.double()[a.long()] - 1), alpha * b.double()[a.long()]
    want = ge * x.double() + be
    # three roundings of the folded gamma, one of beta, one fused multiply-add
    tol = 2.0 ** -23 * (2 * (1 + 2 * ge.abs()) * x.double().abs() + be.abs() + want.abs()) + 1e-30
    assert ((out.double() - want).abs() <= tol).all()
