"""Accuracy of the anchor block's eigendecomposition, seen through handles whose points are their anchors: W W^T = K_SS, the
columns of W are orthogonal, and the eigenvalues add up to the trace."""
import numpy as np
import pytest
import torch

from oracle import kernel as ok

pytestmark = pytest.mark.gpu


def _handle(gpu_lib, X, eps, prec):
    k = len(X)
    P = gpu_lib.Preconditioner(torch.from_numpy(X), eps, [1e-3], k, anchors=torch.arange(k), prec=prec)
    assert P.info()["kept"] == k
    return np.array(P.info()["lam"]), P.get(P.W64).cpu().numpy()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("k,eps", [(150, 1 / 25), (150, 1 / 28), (500, 1 / 28)])
def test_points_far_apart(gpu_lib, k, eps, prec):
    """K_SS = I + entries of 1e-11 and less: every cosine is small from the start, and so is every gap."""
    g = np.stack(np.meshgrid(*[np.arange(8.0)] * 3, indexing="ij"), -1).reshape(-1, 3)[:k]
    X = g + 0.02 * np.random.default_rng(k).standard_normal(g.shape)
    lam, W = _handle(gpu_lib, X, eps, prec)
    M = W.T @ W
    cos = M / np.sqrt(np.outer(np.diag(M), np.diag(M))) - np.eye(k)
    # the sweeps end at cosines of 1e-13; a product of k terms adds some tens of roundings
    assert np.abs(cos).max() <= 2e-13 + 0.2 * k * 2.0 ** -52
    np.testing.assert_allclose(W @ W.T, ok.kernel_matrix(X, X, eps), rtol=0, atol=1e-13 + k * 2.0 ** -52)


@pytest.mark.parametrize("k,d,eps", [(150, 3, 0.05), (700, 3, 0.004), (1000, 4, 0.02)])
def test_rotations_keep_norms(gpu_lib, k, d, eps):
    """FP64 handles: thousands of rotations of a column, each off by half a unit in its cosine and sine, add up like a random
    walk: 20 sweeps of k steps, 2 (20 k)^(1/2) 2^-53 for a column, less for their sum."""
    X = np.random.default_rng(k).random((k, d))
    lam, W = _handle(gpu_lib, X, eps, "fp64")
    walk = 2 * np.sqrt(20.0 * k) * 2.0 ** -53
    assert abs(lam.sum() - k) <= walk * k
    # entries of W W^T: sums of k products with a walk each, and the kernel's own roundings (32 of them)
    np.testing.assert_allclose(W @ W.T, ok.kernel_matrix(X, X, eps), rtol=0, atol=2 * walk + (np.sqrt(k) + 32) * 2.0 ** -53)


def test_rotations_by_single_rows(gpu_lib):
    """More than 4800 anchors, mixed: the accumulated rotations are applied to one row at a time (four no longer fit in LDS)."""
    k = 4810
    X = np.random.default_rng(0).random((k, 8))
    lam, W = _handle(gpu_lib, X, 0.05, "mixed")
    rows = np.random.default_rng(1).choice(k, 300, replace=False)
    K = ok.kernel_matrix(X[rows], X, 0.05)
    # as above, with the operations of this form each rounded: 20 sweeps, three roundings a step and no mean of zero
    assert abs(lam.sum() - k) <= 20 * k * 2.0 ** -53 * k
    np.testing.assert_allclose(W[rows] @ W.T, K, rtol=0, atol=20 * k * 2.0 ** -53)
