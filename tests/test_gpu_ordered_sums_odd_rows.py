"""Segmented sums over rows ordered by cluster on fp32 rows of an odd length (a lane's two channels lie 64 apart), and the
seeded initial rows when many draws collide, against double-precision torch / the host walk."""
import pytest
import torch

from paper_2509_26277_amd import binding, cat_fit, cat_stats, cat_update

pytestmark = pytest.mark.gpu


# rows of 1 .. 17 slices of 128 channels with 1, 63, 64, 65, 127 channels in the last; at least 2^22 elements take the ordered sums
@pytest.mark.parametrize("N,D,K", [(4200000, 1, 3), (66600, 63, 5), (65600, 65, 7), (34000, 127, 4), (33000, 129, 40),
                                   (22001, 193, 6), (4300, 1001, 200), (2100, 2049, 9), (9999, 511, 1)])
def test_sums_and_statistics_on_odd_rows(N, D, K):
    g = torch.Generator(device="cuda")
    g.manual_seed(N + D)
    a = torch.randint(0, K, (N,), generator=g, device="cuda", dtype=torch.int32)
    if K > 3:
        a[a == 2] = 1  # an empty cluster
    x = torch.randn(N, D, generator=g, device="cuda") + a[:, None]
    y = 1.5 * x + 0.3 * torch.randn(N, D, generator=g, device="cuda")
    h = torch.nn.functional.one_hot(a.long(), K).double().t()
    n = h.sum(1).clamp(min=1)[:, None]
    xd, yd = x.double(), y.double()
    mx, my = h @ xd / n, h @ yd / n
    prev = torch.full((K, D), 7.0, device="cuda")
    cent, counts = cat_update(x, a, prev)
    empty = h.sum(1) == 0
    want = torch.where(empty[:, None], prev.double(), mx)
    assert torch.equal(counts.double(), h.sum(1))
    assert ((cent.double() - want).abs() <= 1e-6 * want.abs().clamp(min=1)).all()  # one float32 rounding of a double sum
    dx, dy = xd - mx[a.long()], yd - my[a.long()]
    var, cov = h @ (dx * dx) / n, h @ (dx * dy) / n
    gw = torch.where(empty[:, None], torch.ones_like(var), cov / var.clamp(min=1e-8))
    bw = torch.where(empty[:, None], torch.zeros_like(var), my - gw * mx)
    gamma, beta, _ = cat_stats(x, y, a, K)
    # float32 shifts and results, double sums: a few 1e-6 of the size of the terms
    assert ((gamma.double() - gw).abs() <= 1e-5 * gw.abs().clamp(min=1)).all()
    assert ((beta.double() - bw).abs() <= 1e-5 * (my.abs() + (gw * mx).abs()).clamp(min=1)).all()


@pytest.mark.parametrize("N,K,seed", [(200, 200, 1), (1003, 1000, 2), (64, 64, 3), (65, 1, 4), (70000, 257, 5), (3, 3, 6), (130, 65, 7)])
def test_initial_rows_with_many_collisions(N, K, seed):
    x = torch.arange(N * 4, device="cuda", dtype=torch.float32).reshape(N, 4)
    r = cat_fit(x, x, K, 0, seed=seed)
    idx = binding.cat_init_indices(N, K, seed)
    assert torch.equal(r["centroids"], x[torch.tensor(idx, device="cuda")])
