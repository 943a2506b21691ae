"""One preconditioned column, where an iteration's vector kernels share their passes: against a dense solve, at the edges
of its row blocks (32 rows, 256 rows) and of the two reductions of W^T r (up to 32768 partial sums and 256 columns), by
both drivers; at the largest size with a residual computed apart."""
import numpy as np
import pytest
import torch

from oracle import kernel as ok

pytestmark = pytest.mark.gpu


def _solve(gpu_lib, X, y, eps, beta, k, prec, mode, replace):
    Xd, yd = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    gpu_lib.set_pcg_mode(mode)
    try:
        P = gpu_lib.Preconditioner(Xd, eps, [beta], k, anchors="fps", prec=prec)
        a, its, rel, _, status = gpu_lib.pcg_solve(Xd, yd, eps, beta, P, tol=1e-10, maxit=500, replace_every=replace,
                                                   prec=prec)
    finally:
        gpu_lib.set_pcg_mode(-1)
    return a.cpu().numpy(), its, rel[0], status


@pytest.mark.parametrize("prec,replace", [("fp64", 0), ("mixed", 5)])
@pytest.mark.parametrize("n,d,k", [(33, 2, 5), (257, 3, 40), (1024, 3, 130), (2049, 4, 200), (2300, 8, 520), (1500, 16, 1100)])
def test_matches_dense_solve(gpu_lib, n, d, k, prec, replace):
    rng = np.random.default_rng(n)
    X, y, eps, beta = rng.random((n, d)), rng.standard_normal(n), 0.2 * d, 0.5
    K = np.exp(-((X[:, None, :] - X[None, :, :]) ** 2).sum(-1) / eps)
    ref = np.linalg.solve(K + beta * np.eye(n), y)
    host, its, rel, status = _solve(gpu_lib, X, y, eps, beta, k, prec, 0, replace)
    graph, gits, grel, gstatus = _solve(gpu_lib, X, y, eps, beta, k, prec, 1, replace)
    np.testing.assert_array_equal(host, graph)
    assert (its, rel, status) == (gits, grel, gstatus)
    # the residual reported is the true one (mixed: with nearly all of K in the preconditioner the products' rounding may
    # keep the recurrence from its tolerance, and the best iterate is returned)
    true = np.linalg.norm(y - K @ host - beta * host) / np.linalg.norm(y)
    assert abs(true - rel) <= 1e-10
    assert status == 0 or prec == "mixed"
    # ||K_beta^{-1}|| <= 1 / beta: a residual of rel ||y|| is an error of rel ||y|| / beta at most
    assert np.linalg.norm(host - ref) <= 2 * max(1e-10, rel) * np.linalg.norm(y) / beta


@pytest.mark.parametrize("n", [32768, 32769])
def test_residual_at_the_largest_size(gpu_lib, n):
    rng = np.random.default_rng(n)
    X, y = rng.random((n, 4)), rng.standard_normal(n)
    a, _, rel, _ = _solve(gpu_lib, X, y, 2.0, 1.0, 300, "mixed", -1, 10)
    rows = rng.integers(0, n, 200)
    r = y[rows] - ok.kernel_mv_rows(X, 2.0, a, rows, shift=1.0)
    assert np.linalg.norm(r) <= 2 * max(1e-10, rel) * np.linalg.norm(y)   # some rows of it
