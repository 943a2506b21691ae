"""Dense factorisations of the preconditioner build at the edges of their tiles: the block Jacobi EVD (8-column blocks,
16-row tiles, 4 / 8 / 16 waves), the blocked Cholesky (64-column panels) and the triangular inverse, through
preconditioners on given anchors."""
import numpy as np
import pytest
import torch

from oracle import kernel as ok
from oracle import precond as op

pytestmark = pytest.mark.gpu


# k around one column, a block pair (8, 16), the panel (64), the wave counts' limits (256, 512) and beyond
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("k", [1, 2, 8, 9, 17, 63, 64, 65, 129, 255, 257, 513, 700])
def test_factor_and_core(gpu_lib, k, prec):
    n, d, eps, beta = 1000, 3, 0.004, 1e-2   # K_SS well conditioned for random anchors at every k
    rng = np.random.default_rng(100 + k)
    X = rng.random((n, d))
    S = np.ascontiguousarray(rng.permutation(n)[:k])
    P = gpu_lib.Preconditioner(torch.from_numpy(X), eps, [beta], k, anchors=torch.from_numpy(S), prec=prec)
    nf = op.nystrom_factor(X, S, eps)
    info = P.info()
    assert info["kept"] == nf["kept"] == k
    np.testing.assert_allclose(info["lam"], np.sort(nf["lam"]), rtol=1e-9, atol=1e-12 * max(info["lam"]))
    W = P.get(P.W64).cpu().numpy()
    np.testing.assert_allclose(W @ W.T, nf["W"] @ nf["W"].T, rtol=0, atol=1e-9)
    L = P.get(P.LCORE, 0).cpu().numpy().T   # column-major storage
    np.testing.assert_allclose(L @ L.T, beta * np.eye(k) + W.T @ W, rtol=1e-12, atol=1e-10)
    assert np.array_equal(L, np.tril(L))
    # the apply goes through the inverse core: (beta I + W W^T) z = x, with the factor the apply uses
    x = rng.standard_normal(n)
    z = P.apply(torch.from_numpy(x)).cpu().numpy()
    Wa = W if prec == "fp64" else P.get(P.W32).cpu().numpy().astype(np.float64)
    res = beta * z + Wa @ (Wa.T @ z) - x
    # ||core|| <= 1 / beta and ||W||^2 <= lam_max(K): a relative residual of a few n u ||W||^2 / beta
    bound = 64 * 1e-16 * n * (np.linalg.norm(Wa, 2) ** 2 / beta + 1)
    assert np.linalg.norm(res) <= bound * np.linalg.norm(x)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_singular_anchor_block(gpu_lib, prec):
    """Repeated points among the anchors: K_SS is exactly singular, and the factor is that of the distinct points."""
    n, d, eps, k = 600, 3, 0.02, 80
    rng = np.random.default_rng(9)
    X = rng.random((n, d))
    S = np.ascontiguousarray(rng.permutation(n)[:k])
    X[S[10:20]] = X[S[:10]]
    P = gpu_lib.Preconditioner(torch.from_numpy(X), eps, [1e-2], k, anchors=torch.from_numpy(S), prec=prec)
    info = P.info()
    assert info["kept"] == k - 10
    distinct = np.concatenate([S[:10], S[20:]])
    nf = op.nystrom_factor(X, distinct, eps)
    W = P.get(P.W64).cpu().numpy()
    np.testing.assert_allclose(W @ W.T, nf["W"] @ nf["W"].T, rtol=0, atol=1e-9)
    lam = np.linalg.eigvalsh(ok.kernel_matrix(X[S], X[S], eps))
    np.testing.assert_allclose(info["lam"], lam, rtol=1e-9, atol=1e-12 * lam.max())
