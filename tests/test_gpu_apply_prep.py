"""The launch that prepares a call of inference (operand, norms, folded parameters): K x D around a whole number of its
workgroups, row lengths around its batches of loads, and the same labels as cat_assign.  With so few rows cat_apply takes a
kernel that needs no preparation, so every shape runs on one that does as well, named in the table (2 the row-tile kernel, 3 the
one that streams the centroids, 1 the tile kernel)."""
import pytest
import torch

from paper_2509_26277_amd import cat_apply, cat_assign

from parity_util import without_few_rows_kernel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("alpha", [0.6, 1.0, 0.0])
@pytest.mark.parametrize("N,D,K,kernel", [(1, 4, 1, 2), (40, 32, 32, 2), (40, 33, 31, 2), (40, 41, 25, 2), (70, 1000, 50, 2),
                                          (70, 1000, 50, 3), (130, 1024, 17, 2), (20, 1028, 16, 1), (200, 512, 128, 2), (300, 384, 200, 3),
                                          (70, 7, 64, 2)])
def test_inference_against_doubles(N, D, K, kernel, alpha):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N + D * K)
    r = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    N = max(N, K)
    cent, g, b = r(K, D), r(K, D), r(K, D)
    x = (cent[torch.arange(N, device="cuda") % K] + 0.1 * r(N, D)).contiguous()
    d = ((x.double()[:, None, :] - cent.double()[None]) ** 2).sum(2)
    labels = d.argmin(1)  # (well separated)
    ge, be = 1 + alpha * (g.double()[labels] - 1), alpha * b.double()[labels]
    want = ge * x.double() + be
    # three roundings of the folded gamma, one of beta, one fused multiply-add
    tol = 2.0 ** -23 * (2 * (1 + 2 * ge.abs()) * x.double().abs() + be.abs() + want.abs()) + 1e-30
    call = lambda: cat_apply(x, cent, g, b, alpha=alpha)
    for out, a in (without_few_rows_kernel(call, (kernel,))[1], call()):
        assert torch.equal(a.long(), labels)
        assert torch.equal(a, cat_assign(x, cent)[0])
        assert ((out.double() - want).abs() <= tol).all()
