"""Eigenvectors from the two-sided factorisation of the tridiagonal matrix, and eigenvalues from its leading minors: spectra on
which pivots vanish, couplings are zero, vectors decay past the range of a double, and eigenvalues lie on either side of the
gap below which the pivoted elimination takes over.

Bounds: an eigenvalue is within a few D eps |C| (the covariance is summed in double); a row of the result satisfies
C v = lambda v to the rounding of its float32 entries (6e-8 |C|) and the rows are at right angles to the same: two of unit length whose entries are each off by 2^-24 of themselves, to 1.2e-7."""
import numpy as np
import pytest
import torch

from paper_2509_26277_amd import cat_pca_fit

pytestmark = pytest.mark.gpu


def _rows(C):
    """2 D rows whose covariance is C: the columns of a square root and their negatives, scaled."""
    w, q = np.linalg.eigh(C)
    r = (q * np.sqrt(np.maximum(w, 0.0))).T * np.sqrt(len(w))
    return np.ascontiguousarray(np.concatenate([r, -r]), dtype=np.float32)


def _check(x, p, right=1e-6):
    D = x.shape[1]
    mean, comps, evals = cat_pca_fit(torch.from_numpy(x).cuda(), p)
    xd = x.astype(np.float64) - x.astype(np.float64).mean(0)
    C = xd.T @ xd / len(x)
    w = np.linalg.eigvalsh(C)[::-1]
    v, lam = comps.cpu().numpy().astype(np.float64), evals.cpu().numpy()
    norm = max(np.abs(w).max(), 1e-300)
    slack = 30 * D * np.finfo(np.float64).eps * norm
    assert np.isfinite(v).all()
    assert np.abs(lam - w[:p]).max() <= slack
    assert np.abs(v @ v.T - np.eye(p)).max() <= right
    assert np.linalg.norm(v @ C - lam[:, None] * v, axis=1).max() <= 3e-7 * norm + slack


@pytest.mark.parametrize("gap", [1e-3, 1e-4, 1e-5, 3e-6, 1.2e-6, 1e-7, 1e-9, 1e-11, 1e-14, 0.0])
def test_pairs_of_close_eigenvalues(gap):
    """rows +-s_j h_j and +-t_j h_j on the columns of a Hadamard matrix, which float32 holds exactly: eigenvalues in pairs whose
    members differ by t^2 alone"""
    h = np.ones((1, 1))
    while len(h) < 128:
        h = np.block([[h, h], [h, -h]])
    s = np.repeat(np.linspace(3.0, 1.0, 64), 2).astype(np.float32)
    t = s * np.sqrt(gap) * (np.arange(128) % 2)
    x = np.concatenate([s[:, None] * h, -s[:, None] * h, t[:, None] * h, -t[:, None] * h])
    _check(np.ascontiguousarray(x, dtype=np.float32), 40, 2e-7)


@pytest.mark.parametrize("step", [2e-5, 5e-6, 2e-6, 5e-7])
def test_a_run_of_eigenvalues_a_step_apart(step):
    """every gap among the first vectors near the one (1e-6) below which they are made orthogonal, on either side: rows +-s_j h_j on
    the columns of a Hadamard matrix, eigenvalues s_j^2"""
    h = np.ones((1, 1))
    while len(h) < 256:
        h = np.block([[h, h], [h, -h]])
    s = np.float32(1.0) + np.arange(256, dtype=np.float32) * np.float32(step)
    x = s[:, None] * h
    _check(np.ascontiguousarray(np.concatenate([x, -x]), dtype=np.float32), 60, 2e-7)


@pytest.mark.parametrize("D", [7, 8, 9, 16, 17, 64, 127, 129, 1000])
def test_tridiagonal_covariances(D):
    """the reflections do nothing; constant diagonals make every other pivot vanish at the centre of the spectrum"""
    t = 2.0 * np.eye(D) + np.eye(D, k=1) * 0.9 + np.eye(D, k=-1) * 0.9
    _check(_rows(t), min(D, 12))


def test_blocks_without_coupling_and_vectors_that_decay():
    D = 260
    d = np.concatenate([np.linspace(9, 8, 20), np.full(40, 0.01), np.linspace(7, 3, 200)])
    off = np.full(D - 1, 1e-3)
    off[::13] = 0.0
    _check(_rows(np.diag(d) + np.diag(off, 1) + np.diag(off, -1)), 30)


def test_a_block_of_equal_entries_and_channels_that_never_move():
    rng = np.random.default_rng(5)
    x = rng.standard_normal((300, 120)).astype(np.float32)
    x[:, 30:60] = 1.5  # constant
    x[:, 60:90] = x[:, :30]  # repeated
    _check(x, 50)
