"""The inference kernel for few rows (one launch, direct-form distances) against the direct-form double-precision kernel:
rows around the sizes where the rows per workgroup change, clusters around a wave's share and a round of loads, row lengths
around a round of channels and not whole groups, both row types, ties, distances that overflow or are no numbers."""
import pytest
import torch

from paper_2509_26277_amd import binding, cat_apply, cat_apply_static

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _automatic_after():
    yield
    binding.debug_apply_kernel(0)
    binding.select_path(binding.CAT_PATH_AUTO)


def _case(N, D, K, dtype, spread=1.0):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N * 7 + D * 3 + K)
    r = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    cent, g, b = spread * r(K, D), r(K, D), r(K, D)
    x = (cent[torch.arange(N, device="cuda") % K] + r(N, D)).to(dtype).contiguous()
    return x, cent.contiguous(), g, b


def _both(x, cent, g, b, alpha):
    binding.debug_apply_kernel(4)
    out, a = cat_apply(x, cent, g, b, alpha=alpha)
    binding.debug_apply_kernel(0)
    binding.select_path(binding.CAT_PATH_STREAM)
    want, wa = cat_apply(x, cent, g, b, alpha=alpha)
    binding.select_path(binding.CAT_PATH_AUTO)
    return out, a, want, wa


SHAPES = [(1, 1, 1), (3, 3, 2), (255, 4, 7), (256, 255, 8), (257, 256, 9), (300, 1001, 50), (512, 257, 63), (513, 1000, 64),
          (1023, 70, 65), (1024, 1024, 16), (1025, 2048, 5), (260, 516, 129), (700, 33, 256), (257, 8192, 3), (2500, 1030, 20)]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("N,D,K", SHAPES)
def test_against_direct_form_doubles(N, D, K, dtype):
    if dtype == torch.bfloat16 and D % 2:
        D += 1
    N = max(N, K)
    for spread, alpha in ((1.0, 0.6), (0.02, 1.0)):
        x, cent, g, b = _case(N, D, K, dtype, spread)
        out, a, want, wa = _both(x, cent, g, b, alpha)
        # the labels are those of sums of the same doubles in another order: D additions of rounding 2^-53 may move a tie
        same = a == wa
        if not bool(same.all()):
            bad = (~same).nonzero()[:, 0]
            da = ((x[bad].double() - cent[a[bad].long()].double()) ** 2).sum(1)
            dw = ((x[bad].double() - cent[wa[bad].long()].double()) ** 2).sum(1)
            assert ((da - dw).abs() <= 2.0 ** -52 * D * torch.maximum(da, dw)).all()
        assert torch.equal(out[same], want[same])  # one fused multiply-add per entry on the same folded parameters


@pytest.mark.parametrize("N,D,K", [(600, 37, 300), (513, 36, 512), (1100, 36, 513), (1100, 36, 1024)])
def test_more_clusters_than_the_automatic_selection_sends_it(N, D, K):
    """the sums of all clusters of a workgroup's rows lie in LDS: fewer rows per workgroup where they would not fit"""
    x, cent, g, b = _case(N, D, K, torch.float32)
    out, a, want, wa = _both(x, cent, g, b, 0.6)
    assert torch.equal(a, wa) and torch.equal(out, want)  # (separated by far more than any rounding)


def test_exact_ties_go_to_the_lowest_index():
    cent = torch.randint(-3, 4, (40, 36), device="cuda").float()
    cent[25:] = cent[:15]
    x = cent[torch.arange(200, device="cuda") % 40] + torch.randint(-1, 2, (200, 36), device="cuda").float()
    beta = torch.arange(40, device="cuda").float()[:, None].expand(40, 36).contiguous()
    binding.debug_apply_kernel(4)
    _, a = cat_apply(x, cent, torch.ones_like(cent), beta)
    d = ((x.double()[:, None] - cent.double()[None]) ** 2).sum(2)  # exact
    assert torch.equal(a.long(), torch.stack([(r == r.min()).nonzero()[0, 0] for r in d]))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("D", [2, 64, 66, 510, 512, 514, 1024, 1030, 2060])
def test_near_ties_are_decided_in_doubles(D, dtype):
    """clusters a rounding error apart, around a round of channels of the exact distance"""
    K, N = 24, 300
    x, cent, g, b = _case(N, D, K, dtype)
    cent = (cent[:1] * (1 + 1e-6 * torch.randn(K, D, device="cuda"))).contiguous()
    x = (cent[:1] + torch.randn(N, D, device="cuda")).to(dtype).contiguous()
    out, a, want, wa = _both(x, cent, g, b, 0.6)
    d = ((x.double()[:, None] - cent.double()[None]) ** 2).sum(2)
    best, got = d.min(1).values, d.gather(1, a.long()[:, None])[:, 0]
    assert (got - best <= 2.0 ** -52 * D * best).all()  # the order of the sums of doubles, no more
    same = a == wa
    assert same.float().mean() > 0.9 and torch.equal(out[same], want[same])


@pytest.mark.parametrize("D", [36, 37])
def test_overflow_and_no_numbers(D):
    x, cent, g, b = _case(70, D, 11, torch.float32)
    x[3] = 3e38
    x[4, 5] = float("nan")
    x[5, 1] = float("inf")
    x[6] *= 1e-30
    cent[0, 2] = float("nan")
    cent[7] = -3e38
    binding.debug_apply_kernel(4)
    out, a = cat_apply(x, cent, g, b, alpha=0.5)
    assert ((a >= 0) & (a < 11)).all()
    d = ((x.double()[:, None] - cent.double()[None]) ** 2).sum(2)
    d[:, 0] = float("inf")
    rows = torch.isfinite(x).all(1)
    assert torch.equal(a[rows].long(), d.argmin(1)[rows])


def test_default_selection_takes_it_without_a_workspace_and_under_capture():
    x, cent, g, b = _case(300, 1000, 50, torch.float32)
    binding.select_path(binding.CAT_PATH_STREAM)
    want, wa = cat_apply(x, cent, g, b, alpha=0.6)
    binding.select_path(binding.CAT_PATH_AUTO)
    out = torch.empty_like(x)
    a = torch.empty(300, dtype=torch.int32, device="cuda")
    cat_apply_static(x, cent, g, b, alpha=0.6, out=out, assignments=a)
    assert torch.equal(out, want) and torch.equal(a, wa)
    # the only kernel that leaves the workspace alone: the others fold the coefficient into parameters of their own there
    ws = torch.full((binding.cat_apply_workspace_bytes(300, 1000, 50),), 0xA5, dtype=torch.uint8, device="cuda")
    out, a = cat_apply(x, cent, g, b, alpha=0.6, workspace=ws)
    assert torch.equal(out, want) and torch.equal(a, wa) and bool((ws == 0xA5).all())
    for which in (1, 2, 3):
        binding.debug_apply_kernel(which)
        cat_apply(x, cent, g, b, alpha=0.6, workspace=ws)
        assert not bool((ws == 0xA5).all())
        ws.fill_(0xA5)
    binding.debug_apply_kernel(0)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        go, ga = cat_apply(x, cent, g, b, alpha=0.6, workspace=ws)
    for seed in range(3):
        x2, _, _, _ = _case(300, 1000, 50, torch.float32, spread=1.0 + seed)
        x.copy_(x2)
        graph.replay()
        binding.select_path(binding.CAT_PATH_STREAM)
        want, wa = cat_apply(x, cent, g, b, alpha=0.6)
        binding.select_path(binding.CAT_PATH_AUTO)
        torch.cuda.synchronize()
        assert torch.equal(go, want) and torch.equal(ga, wa) and bool((ws == 0xA5).all())


def test_a_shape_it_does_not_take_is_an_error():
    x, cent, g, b = _case(40, 8200, 3, torch.float32)
    binding.debug_apply_kernel(4)
    with pytest.raises(binding.CatError) as e:
        cat_apply(x, cent, g, b)
    assert e.value.status == 2
