"""The PCA front-end on short rows: column sums and covariance of up to 64 (256) columns in few workgroups, the tridiagonalisation
below 64 in one workgroup, and the projection that leaves out the steps past the end of a row.

Bounds.  Mean and covariance are summed in double on both sides: they, and with them the eigenvalues, differ by N eps and D eps of their
scale.  A score is a sum of D products in fp32: D + 2 roundings of at most the sum of their magnitudes."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_26277_amd import binding, cat_apply_pca, cat_pca_fit, cat_pca_project

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps


def _rows(N, D, dtype):
    rng = np.random.default_rng(1000 * N + D)
    x = torch.from_numpy((rng.standard_normal((N, D)) * np.linspace(3.0, 0.5, D) + rng.standard_normal(D)).astype(np.float32))
    x = x.bfloat16() if dtype == "bf16" else x
    return x.cuda(), x.float().numpy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N,D", [
    (1, 5), (31, 15), (33, 16), (255, 17), (257, 31), (600, 32), (1000, 33), (513, 47), (511, 48), (2049, 49), (5000, 62), (70001, 63),
    (4096, 64), (90001, 30), (300, 65), (5000, 128), (3000, 129), (2000, 255), (20001, 256), (1500, 257),
])
def test_pairs_of_the_covariance(N, D, dtype):
    lq, x = _rows(N, D, dtype)
    p = min(D, 9)
    mean, comps, evals = cat_pca_fit(lq, p)
    mean_o, C = oracle.covariance(x)
    w = np.linalg.eigvalsh(C)[::-1][:p]
    v, lam = comps.cpu().numpy().astype(np.float64), evals.cpu().numpy()
    scale = np.abs(x.astype(np.float64)).max()
    np.testing.assert_allclose(mean.cpu().numpy(), mean_o, rtol=6e-8, atol=N * EPS * scale + 1e-30)
    norm = max(w[0], 1e-300)
    slack = (30 * D + N) * EPS * max(norm, 1e-30) + N * EPS * (EPS * scale**2)
    assert np.abs(lam - w).max() <= slack
    assert np.abs(v @ v.T - np.eye(p)).max() <= 1e-6
    assert np.linalg.norm(v @ C - lam[:, None] * v, axis=1).max() <= 3e-7 * norm + slack


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N,D,p", [(100, 20, 17), (129, 60, 50), (64, 64, 64), (200, 112, 33), (200, 116, 20), (77, 128, 30), (90, 132, 34),
                                   (130, 196, 49), (300, 252, 70), (128, 260, 18), (50, 24, 10)])
def test_scores_of_rows_that_end_inside_a_chunk(N, D, p, dtype):
    lq, x = _rows(N, D, dtype)
    rng = np.random.default_rng(D + p)
    mean = rng.standard_normal(D).astype(np.float32)
    comps = rng.standard_normal((p, D)).astype(np.float32)
    z = cat_pca_project(lq, torch.from_numpy(mean).cuda(), torch.from_numpy(comps).cuda()).cpu().numpy()
    d = x.astype(np.float64) - mean
    bound = (D + 2) * 2.0**-24 * (np.abs(d) @ np.abs(comps.astype(np.float64)).T)
    assert (np.abs(z - d @ comps.T.astype(np.float64)) <= bound).all()


@pytest.mark.parametrize("D,p,dtype", [(72, 20, "f32"), (136, 32, "f32"), (344, 25, "f32"), (124, 17, "bf16"), (640, 30, "bf16")])
def test_fused_inference_with_many_rows(D, p, dtype):
    """17 .. 32 directions: above 65536 rows the steps past a row's end may be done, on zeros: the same bits as without them"""
    g = torch.Generator(device="cuda").manual_seed(D)
    N, K = 66003, 7
    lq = torch.randn(N, D, generator=g, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    mean, comps = torch.randn(D, generator=g, device="cuda"), torch.randn(p, D, generator=g, device="cuda") / D ** 0.5
    cz = torch.randn(K, p, generator=g, device="cuda")
    gamma, beta = torch.rand(K, D, generator=g, device="cuda") + 0.5, torch.randn(K, D, generator=g, device="cuda")
    out, a = cat_apply_pca(lq, mean, comps, cz, gamma, beta, alpha=0.7)
    few, b = cat_apply_pca(lq[:65536], mean, comps, cz, gamma, beta, alpha=0.7)
    assert torch.equal(a[:65536], b) and torch.equal(out[:65536], few)
    try:
        binding.select_path(binding.CAT_PATH_STREAM)
        steps, c = cat_apply_pca(lq, mean, comps, cz, gamma, beta, alpha=0.7)
    finally:
        binding.select_path(binding.CAT_PATH_AUTO)
    assert torch.equal(a, c) and torch.equal(out, steps)


@pytest.mark.parametrize("N,D,p", [(301, 512, 64), (129, 1000, 33), (32768, 120, 50), (32769, 120, 50), (700, 104, 40)])
def test_fused_inference_equals_the_steps_either_side_of_its_lines(N, D, p):
    """33 .. 64 directions on fp32 rows: with the steps past a row's end (few of them, few rows) and without"""
    g = torch.Generator(device="cuda").manual_seed(N + D)
    K = 9
    lq = torch.randn(N, D, generator=g, device="cuda")
    mean, comps = torch.randn(D, generator=g, device="cuda"), torch.randn(p, D, generator=g, device="cuda") / D ** 0.5
    cz = torch.randn(K, p, generator=g, device="cuda")
    gamma, beta = torch.rand(K, D, generator=g, device="cuda") + 0.5, torch.randn(K, D, generator=g, device="cuda")
    out, a = cat_apply_pca(lq, mean, comps, cz, gamma, beta, alpha=0.7)
    try:
        binding.select_path(binding.CAT_PATH_STREAM)
        steps, c = cat_apply_pca(lq, mean, comps, cz, gamma, beta, alpha=0.7)
    finally:
        binding.select_path(binding.CAT_PATH_AUTO)
    assert torch.equal(a, c) and torch.equal(out, steps)
