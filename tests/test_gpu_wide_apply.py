"""Inference with the streamed centroid operand (cat_wide_kernel.h): edges of its instances (steps per wave, cluster tiles,
rows per tile), rows that are not whole 16-byte groups, near-ties and exact ties, against double-precision torch."""
import pytest
import torch

from paper_2509_26277_amd import binding, cat_apply

pytestmark = pytest.mark.gpu


def _exact(x, cent, g, b, alpha):
    xd, c = x.double(), cent.double()
    d = torch.cat([((r[:, None, :] - c[None]) ** 2).sum(2) for r in xd.split(64)])
    two = d.topk(min(2, d.shape[1]), 1, largest=False).values
    lowest = torch.where(d == two[:, :1], torch.arange(d.shape[1], device="cuda"), d.shape[1]).min(1).values
    return lowest, d, xd + alpha * (g.double()[lowest] * xd + b.double()[lowest] - xd)


def _check(x, cent, g, b, alpha, bf16):
    out, a = cat_apply(x, cent, g, b, alpha=alpha)
    want, d, corr = _exact(x, cent, g, b, alpha)
    a = a.long()
    bad = (a != want).nonzero().flatten()
    if len(bad):  # equidistant to the rounding of a double sum
        da, dw = d[bad, a[bad]], d[bad, want[bad]]
        assert ((da - dw) <= 1e-12 * dw).all(), (bad[:5], a[bad][:5], want[bad][:5])
    ok = a == want
    err = (out.double() - corr).abs()[ok]
    # one fused multiply-add in float32 with parameters folded in float32; bf16 rows are rounded to bf16 once more
    tol = (2.0 ** -8 if bf16 else 4e-7) * corr.abs()[ok] + 2e-6
    assert (err <= tol).all(), float((err - tol).max())
    out2, none = cat_apply(x, cent, g, b, alpha=alpha, want_assignments=False)
    assert none is None and torch.equal(out, out2)
    return a


def _case(seed, N, D, K, bf16, spread=1.0):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    r = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    cent = r(K, D) * spread
    x = cent[torch.randint(0, K, (N,), generator=gen, device="cuda")] + r(N, D)
    x = x.bfloat16() if bf16 else x
    return x.contiguous(), cent.contiguous(), 1.0 + 0.3 * r(K, D), 0.5 * r(K, D)


F32 = [(1, 1000, 50), (1, 1001, 33), (51, 1001, 50), (1, 1023, 64), (65, 1024, 33), (257, 999, 48), (100, 513, 64), (77, 514, 65), (64, 300, 100),
       (129, 512, 128), (65, 511, 128), (130, 129, 128), (500, 255, 70), (97, 257, 64), (40, 1021, 20), (40, 1024, 128), (35, 897, 127)]
BF16 = [(1, 2048, 64), (33, 2046, 64), (95, 2040, 50), (64, 1026, 33), (63, 1024, 64), (257, 1022, 128), (100, 1024, 65), (31, 512, 128),
        (130, 514, 40), (70, 510, 64), (44, 2048, 17), (66, 1536, 20), (200, 130, 100)]


@pytest.mark.parametrize("N,D,K", F32)
def test_fp32_rows(N, D, K):
    x, c, g, b = _case(N + D + K, max(N, K), D, K, False, 0.3)
    _check(x, c, g, b, 0.6, False)


@pytest.mark.parametrize("N,D,K", BF16)
def test_bf16_rows(N, D, K):
    x, c, g, b = _case(N + D + K, max(N, K), D, K, True, 0.3)
    _check(x, c, g, b, 1.0, True)


@pytest.mark.parametrize("N,D,K,bf16", [(200, 1001, 50, False), (200, 1000, 64, False), (200, 2048, 64, True), (200, 2046, 40, True),
                                        (150, 512, 128, False), (150, 1022, 128, True)])
def test_near_and_exact_ties(N, D, K, bf16):
    """repeated centroids (exact ties: the lowest index), up to 8 candidates and beyond, centroids a rounding error apart"""
    x, c, g, b = _case(D, N, D, K, bf16, 0.2)
    for copies in (2, 5, 12):
        c2 = c[: (K + copies - 1) // copies].repeat(copies, 1)[:K].contiguous()
        a = _check(x, c2, g, b, 0.5, bf16)
        assert int(a.max()) < (K + copies - 1) // copies
    c3 = c.clone()
    c3[1::2] = c3[0::2][: len(c3[1::2])] * (1 + 1e-6)
    _check(x, c3.contiguous(), g, b, 0.5, bf16)


@pytest.mark.parametrize("N,D,K,bf16", [(300, 1001, 50, False), (300, 2048, 64, True)])
def test_non_finite_rows_and_many_tiles(N, D, K, bf16):
    x, c, g, b = _case(5, N, D, K, bf16)
    want = cat_apply(x, c, g, b)
    x2 = x.clone()
    x2[3] = float("nan")
    x2[40, 7] = float("inf")
    x2[299, 1] = -float("inf")
    out, a = cat_apply(x2, c, g, b)
    keep = torch.ones(N, dtype=torch.bool, device="cuda")
    keep[[3, 40, 299]] = False
    assert torch.equal(a[keep], want[1][keep]) and torch.equal(out[keep], want[0][keep])
    assert int(a.min()) >= 0 and int(a.max()) < K


@pytest.mark.parametrize("D,K,bf16", [(1001, 50, False), (1000, 50, False), (2048, 64, True), (512, 128, False)])
def test_long_launches_match_the_tile_kernel(D, K, bf16):
    """more tiles than workgroups, against the kernels that take these shapes when told to"""
    x, c, g, b = _case(9, 40000, D, K, bf16, 0.5)
    out, a = cat_apply(x, c, g, b, alpha=0.3)
    try:
        binding.debug_apply_kernel(1)
        out1, a1 = cat_apply(x, c, g, b, alpha=0.3)
    finally:
        binding.debug_apply_kernel(0)
    assert torch.equal(a, a1)
    assert torch.equal(out, out1)


def test_captures_into_a_hip_graph_and_replays():
    x, c, g, b = _case(2, 3000, 1001, 50, False)
    out = torch.empty_like(x)
    ws = torch.empty(binding.cat_apply_workspace_bytes(3000, 1001, 50), dtype=torch.uint8, device="cuda")
    cat_apply(x, c, g, b, alpha=0.6, out=out, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        _, a = cat_apply(x, c, g, b, alpha=0.6, out=out, workspace=ws)
    for seed in (3, 4, 5):
        x2 = _case(seed, 3000, 1001, 50, False)[0]
        x.copy_(x2)
        graph.replay()
        torch.cuda.synchronize()
        o2, a2 = cat_apply(x2, c, g, b, alpha=0.6)
        assert torch.equal(out, o2) and torch.equal(a, a2)
