"""Pivoted QR of columns whose residuals fall by orders of magnitude within a batch, without their rank being exhausted: a
batch ends where its Gram matrix no longer resolves them."""
import numpy as np
import pytest
import scipy.linalg
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n,fall", [(60, 3.0), (900, 20.0), (3000, 8.0)])
def test_graded_columns(gpu_lib, n, fall, prec):
    """Each picked column's residual is `fall` times shorter than the one before, the other columns lie below the shortest."""
    l, k = 40, 40 if fall < 5 else 12
    rng = np.random.default_rng(n)
    Q = np.linalg.qr(rng.standard_normal((l, l)))[0].T
    at = rng.permutation(n)[:k]
    Y = rng.standard_normal((n, l)) * fall ** -(k + 3)
    for j in range(k):   # direction j, and something of those before it
        Y[at[j]] = (Q[j] + 0.3 * rng.standard_normal(j) @ Q[:j] / max(j, 1) ** 0.5) * fall ** -j
    if prec == "fp32":
        Y = Y.astype(np.float32).astype(np.float64)
    piv, rd = gpu_lib.qrcp(torch.from_numpy(Y), k, prec=prec)
    R, order = scipy.linalg.qr(Y.T, mode="r", pivoting=True)
    np.testing.assert_array_equal(order[:k], at)
    np.testing.assert_array_equal(piv.cpu().numpy(), at)
    # a column's squared norm is no more than a tenth above its residual's: downdating keeps some k units of its own
    np.testing.assert_allclose(rd.cpu().numpy(), np.abs(np.diag(R))[:k], rtol=100 * k * 2.0 ** -53, atol=0)
