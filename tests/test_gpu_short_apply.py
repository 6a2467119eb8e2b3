"""Inference over short rows (cat_short.hip): rows of at most 512 bytes, moved as pieces of 16 rows.

Against the oracle in double precision: the ranking is exact (rows whose two nearest centroids tie to 1e-5 are exempt), the map one
fused multiply-add per entry on parameters folded in fp32, bfloat16 results rounded once."""
import threading

import numpy as np
import pytest
import torch

import oracle
from paper_2509_26277_amd import binding, cat_apply

from parity_util import check_assignments_lazy, check_values, dev_matrix, f32_round, host_matrix

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _short_rows():
    binding.debug_apply_kernel(5)  # this kernel or an error
    yield
    binding.debug_apply_kernel(0)


def _case(N, D, K, dtype, seed, spread=2.0):
    rng = np.random.default_rng(seed)
    cent = rng.standard_normal((K, D)) * spread
    x = cent[rng.integers(0, K, N)] + rng.standard_normal((N, D))
    if dtype == "bf16":
        x = torch.from_numpy(x).bfloat16().float().numpy()
    g, b = rng.uniform(0.5, 1.5, (K, D)), rng.standard_normal((K, D))
    return x.astype(np.float32), f32_round(cent), f32_round(g), f32_round(b)


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


def _check(x, cent, g, b, alpha, dtype):
    out, a = cat_apply(dev_matrix(x, dtype), _dev(cent), _dev(g), _dev(b), alpha=alpha)
    a = a.cpu().numpy()
    want, label = oracle.apply(x, cent, g, b, alpha)
    check_assignments_lazy(a, label, x, cent, "labels")
    same = a == label
    # fp32: folding rounds gamma' and beta' (6e-8 each, of 1 + alpha |gamma - 1|), the product once more; bf16: half a unit of 2^-8
    check_values(host_matrix(out)[same], want[same], 1e-6 if dtype == "f32" else 4e-3, "corrected")
    return a


SHAPES = [
    # N, D, K: fewest channels, remainders of 16 rows, whole 16-byte groups and not, each number of groups per lane
    (1025, 4, 1, "f32"), (1030, 5, 2, "f32"), (1039, 7, 16, "f32"), (1040, 31, 17, "f32"), (1100, 32, 33, "f32"), (1337, 33, 5, "f32"),
    (1041, 63, 20, "f32"), (1042, 64, 65, "f32"), (1043, 65, 9, "f32"), (1044, 127, 3, "f32"), (1045, 128, 30, "f32"), (40001, 127, 60, "f32"),
    (40003, 128, 128, "f32"), (33333, 20, 128, "f32"),
    (1025, 8, 1, "bf16"), (1030, 10, 2, "bf16"), (1039, 62, 16, "bf16"), (1040, 64, 17, "bf16"), (1041, 66, 33, "bf16"), (1337, 126, 5, "bf16"),
    (1042, 128, 65, "bf16"), (1043, 130, 9, "bf16"), (1044, 254, 3, "bf16"), (1045, 256, 20, "bf16"), (20001, 250, 16, "bf16"), (20002, 248, 60, "bf16"),
]


@pytest.mark.parametrize("alpha", [1.0, 0.6])
@pytest.mark.parametrize("N,D,K,dtype", SHAPES)
def test_against_the_oracle(N, D, K, dtype, alpha):
    _check(*_case(N, D, K, dtype, N + D + K), alpha, dtype)


def test_near_ties_are_measured():
    """clusters that overlap, far from the origin: many rows within the error bound of the split arithmetic; equal centroids"""
    x, cent, g, b = _case(3000, 45, 12, "f32", 3, spread=0.05)
    x = (x + 30.0).astype(np.float32)
    cent = f32_round(cent + 30.0)
    cent[7] = cent[2]
    a = _check(x, cent, g, b, 0.6, "f32")
    assert not (a == 7).any()  # the lowest of two equal centroids


def test_without_labels_and_other_rows_beside_non_finite_ones():
    x, cent, g, b = _case(2000, 50, 6, "f32", 8)
    x[5] = np.nan
    x[700, 3] = np.inf
    lq = dev_matrix(x, "f32")
    out, a = cat_apply(lq, _dev(cent), _dev(g), _dev(b))
    a = a.cpu().numpy()
    assert ((a >= 0) & (a < 6)).all()
    fine = np.ones(2000, dtype=bool)
    fine[[5, 700]] = False
    want, label = oracle.apply(x[fine], cent, g, b, 1.0)
    assert (a[fine] == label).all()
    check_values(host_matrix(out)[fine], want, 1e-6, "corrected")
    lib = binding.load_library()
    again = torch.full_like(out, 7.0)
    ws = torch.empty(binding.cat_apply_workspace_bytes(2000, 50, 6), dtype=torch.uint8, device="cuda")
    c, gg, bb = _dev(cent), _dev(g), _dev(b)
    assert lib.cat_apply(lq.data_ptr(), 2000, 50, 6, binding.CAT_F32, c.data_ptr(), gg.data_ptr(), bb.data_ptr(), 1.0, again.data_ptr(),
                         None, ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    assert torch.equal(again[:5], out[:5]) and torch.equal(again[701:], out[701:])


@pytest.mark.parametrize("N,D,K,dtype", [(1100, 129, 5, "f32"), (1100, 3, 5, "f32"), (1100, 258, 5, "bf16"), (1100, 6, 5, "bf16"), (1100, 64, 129, "f32"),
                                         (1100, 127, 100, "f32"), (1100, 250, 40, "bf16")])
def test_shapes_outside_are_refused(N, D, K, dtype):
    """longer than 512 bytes, shorter than 16, more than 128 clusters; unaligned rows whose parameters do not fit LDS"""
    x, cent, g, b = _case(N, D, K, dtype, 1)
    with pytest.raises(binding.CatError, match="CAT_ERR_UNSUPPORTED"):
        cat_apply(dev_matrix(x, dtype), _dev(cent), _dev(g), _dev(b))


@pytest.mark.parametrize("N,D,K,dtype", [(4706, 101, 16, "f32"), (5941, 4, 100, "f32"), (2041, 118, 16, "f32"), (6444, 200, 54, "bf16"), (20000, 100, 50, "f32"),
                                         (4096, 32, 10, "f32"), (3000, 120, 70, "bf16"), (12479, 4, 22, "f32"), (3253, 24, 90, "f32"), (3420, 106, 3, "bf16")])
def test_the_dispatch_gives_what_each_kernel_gives(N, D, K, dtype):
    """either side of the rule's lines: the same labels and, to the rounding of a fold, the same rows as the kernel forced"""
    x, cent, g, b = _case(N, D, K, dtype, 2, spread=1.0)
    lq, p = dev_matrix(x, dtype), (_dev(cent), _dev(g), _dev(b))
    forced, a = cat_apply(lq, *p, alpha=0.6)
    binding.debug_apply_kernel(0)
    out, a0 = cat_apply(lq, *p, alpha=0.6)
    assert (a == a0).all()
    check_values(host_matrix(out), host_matrix(forced), 1e-6 if dtype == "f32" else 8e-3, "corrected")


def test_threads_that_use_one_kernel_with_different_amounts_of_lds():
    """one instance, parameters of few and of many channels: what a launch may take is not lowered by a smaller one beside it"""
    cases = [_case(3000, D, K, "f32", D, spread=1.0) for D, K in ((36, 17), (64, 32))]
    dev = [(dev_matrix(x, "f32"), _dev(c), _dev(g), _dev(b)) for x, c, g, b in cases]
    want = [cat_apply(*d) for d in dev]
    torch.cuda.synchronize()
    wrong = []

    def work(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(50):
                    out, a = cat_apply(*dev[i])
                    torch.cuda.current_stream().synchronize()
                    if not (torch.equal(out, want[i][0]) and torch.equal(a, want[i][1])):
                        raise AssertionError("other results")
        except Exception as e:
            wrong.append((i, e))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong, wrong
