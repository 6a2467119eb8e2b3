"""The leading eigenpairs behind cat_pca_fit (tridiagonalisation, multisection, inverse iteration) at the sizes where the
kernels change their layout, on spectra with multiple eigenvalues, and against the Jacobi sweeps they replace.

Bounds.  Eigenvalues: the covariance is summed in double on both sides, so they differ by a few D eps |C|.  Directions:
rounded to float32 (6e-8 of a unit vector), and turned by at most (a few D eps |C|) / gap."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_26277_amd import cat_pca_fit

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps


def _check(x, p, **kw):
    D = x.shape[1]
    mean_o, C = oracle.covariance(x)
    w = np.linalg.eigvalsh(C)[::-1]
    mean, comps, evals = cat_pca_fit(torch.from_numpy(x).cuda(), p, **kw)
    v, lam = comps.cpu().numpy().astype(np.float64), evals.cpu().numpy()
    norm = max(np.abs(w).max(), 1e-300)
    slack = 30 * D * EPS * norm
    assert np.isfinite(v).all()
    np.testing.assert_allclose(mean.cpu().numpy(), mean_o, rtol=1e-6, atol=1e-6)
    assert np.abs(lam - w[:p]).max() <= slack
    assert np.abs(v @ v.T - np.eye(p)).max() <= 1e-6  # rows of length 1 at right angles, as float32 holds them
    assert np.linalg.norm(v @ C - lam[:, None] * v, axis=1).max() <= 3e-7 * norm + slack
    big = np.abs(v).max(axis=1)
    for c in range(p):  # the first entry of largest magnitude is positive (near-ties: any of the largest)
        assert v[c][np.abs(v[c]) >= big[c] * (1 - 1e-6)].max() > 0
    return lam, v, w, slack


@pytest.mark.parametrize("D", [1, 2, 3, 5, 8, 9, 63, 64, 65, 255, 256, 257, 264, 511, 513, 769, 777, 1024, 1025, 1537, 2047, 2048])
def test_leading_pairs_at_the_edges_of_the_layouts(D):
    rng = np.random.default_rng(D)
    N, p = 400, min(D, 7)
    x = (rng.standard_normal((N, D)) * np.linspace(3.0, 0.5, D) + rng.standard_normal(D)).astype(np.float32)
    lam, v, w, slack = _check(x, p)
    _, comps_o, _ = oracle.pca_fit(x, p)
    gap = np.array([min(w[i - 1] - w[i] if i else np.inf, w[i] - w[i + 1] if i + 1 < D else np.inf) for i in range(p)])
    for c in range(p):
        assert np.abs(v[c] - comps_o[c]).max() <= 2e-7 + slack / gap[c]


@pytest.mark.parametrize("N,D,p", [(20, 96, 40), (3, 64, 64), (2, 33, 20), (500, 256, 256), (400, 300, 256)])
def test_rank_deficient_and_full(N, D, p):
    """more directions than the rows span: the rest are an orthonormal set of the null space; and the largest p"""
    rng = np.random.default_rng(N + D)
    _check((rng.standard_normal((N, D)) + 0.5).astype(np.float32), p)


@pytest.mark.parametrize("D,p", [(40, 40), (130, 60)])
def test_multiple_eigenvalues(D, p):
    """rows +-s e_j: a diagonal covariance with few distinct values, exactly repeated (the tridiagonal matrix splits)"""
    s = np.where(np.arange(D) % 3 == 0, 4.0, np.where(np.arange(D) % 3 == 1, 2.0, 1.0))
    x = np.concatenate([np.diag(s), -np.diag(s)]).astype(np.float32)
    _check(x, p)


@pytest.mark.parametrize("x", [np.zeros((10, 17)), np.full((5, 70), 3.25), np.tile(np.random.default_rng(1).standard_normal((30, 20)), (1, 5)),
                               np.random.default_rng(2).standard_normal((200, 90)) * 1e-12,
                               np.random.default_rng(3).standard_normal((200, 90)) * 1e12])
def test_constant_repeated_and_scaled_channels(x):
    x = x.astype(np.float32)
    D = x.shape[1]
    lam, v, w, slack = _check(x, min(D, 16))
    assert lam.min() >= -slack


@pytest.mark.parametrize("N,D,p", [(900, 200, 30), (700, 64, 64)])
def test_agrees_with_the_jacobi_sweeps(N, D, p):
    """a number of sweeps given: one-sided Jacobi over all rows; the same eigenpairs"""
    rng = np.random.default_rng(N)
    x = torch.from_numpy((rng.standard_normal((N, D)) * np.linspace(4, 1, D)).astype(np.float32)).cuda()
    m0, c0, l0 = cat_pca_fit(x, p)
    m1, c1, l1 = cat_pca_fit(x, p, sweeps=12)
    assert torch.equal(m0, m1) or (m0 - m1).abs().max() < 1e-6
    assert ((l0 - l1).abs() <= 1e-12 * l1[0]).all()
    assert (c0 - c1).abs().max() <= 1e-5
