"""Inference with the streamed centroid operand (cat_wide_kernel.h): edges of its instances (steps per wave, cluster tiles,
rows per tile), rows that are not whole 16-byte groups, near-ties and exact ties, against double-precision torch.  The shapes
that it has an instance for are run on it whatever cat_apply would choose; the others of each table run as they come, and where
that is the kernel for few rows, on the one that more rows would take too."""
import pytest
import torch

from paper_2509_26277_amd import binding, cat_apply

from parity_util import without_few_rows_kernel

pytestmark = pytest.mark.gpu


def _exact(x, cent, g, b, alpha):
    xd, c = x.double(), cent.double()
    d = torch.cat([((r[:, None, :] - c[None]) ** 2).sum(2) for r in xd.split(64)])
    two = d.topk(min(2, d.shape[1]), 1, largest=False).values
    lowest = torch.where(d == two[:, :1], torch.arange(d.shape[1], device="cuda"), d.shape[1]).min(1).values
    return lowest, d, xd + alpha * (g.double()[lowest] * xd + b.double()[lowest] - xd)


def _has_instance(D, K, bf16):
    """rows of up to 4 KB (K > 128: 3 KB); not the shapes the row-tile kernel always keeps"""
    row = D * (2 if bf16 else 4)
    if bf16:
        rowtile = (K <= 32 and D <= 1024) or (K <= 64 and D <= 512)
    else:
        rowtile = (K <= 32 and D <= 1024) or (K <= 128 and D <= 512)
    return row <= (4096 if K <= 128 else 3072) and not rowtile


@pytest.fixture(autouse=True)
def _automatic_after():
    yield
    binding.debug_apply_kernel(0)


def _check(x, cent, g, b, alpha, bf16):
    if _has_instance(x.shape[1], cent.shape[0], bf16):
        binding.debug_apply_kernel(3)
    else:
        out, a = without_few_rows_kernel(lambda: cat_apply(x, cent, g, b, alpha=alpha), (2, 1))[1]
        _check_one(x, cent, g, b, alpha, bf16, out, a)
    out, a = cat_apply(x, cent, g, b, alpha=alpha)
    a = _check_one(x, cent, g, b, alpha, bf16, out, a)
    out2, none = cat_apply(x, cent, g, b, alpha=alpha, want_assignments=False)
    assert none is None and torch.equal(out, out2)
    return a


def _check_one(x, cent, g, b, alpha, bf16, out, a):
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
       (129, 512, 128), (65, 511, 128), (130, 129, 128), (500, 255, 70), (97, 257, 64), (40, 1021, 20), (40, 1024, 128), (35, 897, 127),
       (300, 514, 64), (300, 768, 60), (300, 767, 64), (300, 769, 40), (300, 516, 128), (300, 765, 100), (300, 1000, 65),
       (200, 300, 129), (260, 301, 200), (256, 512, 256), (300, 255, 255), (200, 520, 129), (260, 701, 200), (256, 768, 256), (300, 767, 250)]
BF16 = [(1, 2048, 64), (33, 2046, 64), (95, 2040, 50), (64, 1026, 33), (63, 1024, 64), (257, 1022, 128), (100, 1024, 65), (31, 512, 128),
        (130, 514, 40), (70, 510, 64), (44, 2048, 17), (66, 1536, 20), (200, 130, 100),
        (64, 1032, 5), (64, 1538, 32), (64, 1030, 16), (90, 1500, 64), (90, 1540, 128), (90, 1498, 100), (90, 1544, 90),
        (200, 700, 129), (260, 702, 200), (256, 1024, 256), (300, 510, 255), (200, 1200, 129), (260, 1202, 200), (256, 1536, 256)]


@pytest.mark.parametrize("N,D,K", F32)
def test_fp32_rows(N, D, K):
    x, c, g, b = _case(N + D + K, max(N, K), D, K, False, 0.3)
    _check(x, c, g, b, 0.6, False)


@pytest.mark.parametrize("N,D,K", BF16)
def test_bf16_rows(N, D, K):
    x, c, g, b = _case(N + D + K, max(N, K), D, K, True, 0.3)
    _check(x, c, g, b, 1.0, True)


@pytest.mark.parametrize("N,D,K,bf16", [(200, 1001, 50, False), (200, 1000, 64, False), (200, 2048, 64, True), (200, 2046, 40, True),
                                        (150, 512, 128, False), (150, 1022, 128, True), (150, 600, 64, False), (150, 768, 128, False),
                                        (300, 512, 256, False), (300, 701, 200, False), (300, 768, 250, False), (300, 1024, 256, True),
                                        (300, 1202, 200, True)])
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


@pytest.mark.parametrize("N,D,K,bf16", [(5000, 1001, 50, False), (5000, 301, 200, False), (5000, 1032, 10, True), (9000, 600, 200, False)])
def test_a_workspace_without_its_operand_is_enough(N, D, K, bf16):
    """the folded parameters alone (what rows that are not whole 16-byte groups need on the streaming kernel), and what the
    tile kernel needs beside them, with and without the scratch of its ranking in two launches"""
    x, c, g, b = _case(3, N, D, K, bf16, 0.5)
    dt = binding.CAT_BF16 if bf16 else binding.CAT_F32
    want = cat_apply(x, c, g, b, alpha=0.6)
    full = binding.cat_apply_workspace_bytes(N, D, K, dt)
    folded = 2 * ((4 * K * D + 255) // 256 * 256)
    sizes = [full - 256, full - 12 * N] if K > 128 else [full - 256]
    if D % (8 if bf16 else 4):
        sizes.append(folded)
    for size in sizes:
        out, a = cat_apply(x, c, g, b, alpha=0.6, workspace=torch.empty(size, dtype=torch.uint8, device="cuda"))
        assert torch.equal(a, want[1]) and torch.equal(out, want[0])
    with pytest.raises(binding.CatError):
        cat_apply(x, c, g, b, alpha=0.6, workspace=torch.empty(folded - 256, dtype=torch.uint8, device="cuda"))


def test_shapes_without_an_instance_are_refused_when_it_is_asked_for():
    for D, K, bf16 in [(1000, 32, False), (512, 128, False), (1025, 100, False), (769, 200, False), (1024, 32, True), (512, 64, True),
                       (1538, 130, True), (2050, 64, True)]:
        assert not _has_instance(D, K, bf16)
        x, c, g, b = _case(1, max(64, K), D, K, bf16)
        binding.debug_apply_kernel(3)
        with pytest.raises(binding.CatError):
            cat_apply(x, c, g, b)


@pytest.mark.parametrize("N,D,K,bf16", [(300, 1001, 50, False), (300, 2048, 64, True), (300, 700, 200, False)])
def test_non_finite_rows_and_many_tiles(N, D, K, bf16):
    x, c, g, b = _case(5, N, D, K, bf16)
    binding.debug_apply_kernel(3)
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


@pytest.mark.parametrize("D,K,bf16", [(1001, 50, False), (1000, 50, False), (2048, 64, True), (512, 128, False), (600, 200, False)])
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
