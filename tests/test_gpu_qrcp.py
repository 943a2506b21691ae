"""Candidate-batch pivoted QR at its edges (candidate set of 1024, batches of 32 steps, 16-column tiles, 4-row quads)
against one pass over the sketch per step (KRR_QR_FULL), and with norms that tie."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _decaying(n, l, seed, decay):
    """Columns (rows of Y) with a generic greedy order: random directions scaled along l."""
    rng = np.random.default_rng(seed)
    return rng.standard_normal((n, l)) * np.exp(-decay * np.arange(l) / l) * (1 + rng.random((n, 1)))


# n: fewer than, exactly and more than the candidate set; l: remainders of 4, 16, 64; k: around the batch, and k = l
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n,l,k", [(1, 1, 1), (40, 33, 33), (300, 67, 31), (1023, 70, 32), (1024, 65, 33), (1025, 129, 64),
                                   (5000, 130, 97), (70001, 45, 45)])
def test_matches_full_pass(gpu_lib, n, l, k, prec, monkeypatch):
    Y = torch.from_numpy(_decaying(n, l, 7 * n + l, 3.0)).cuda()
    piv, rd = gpu_lib.qrcp(Y, k, prec=prec)
    monkeypatch.setenv("KRR_QR_FULL", "1")
    piv_f, rd_f = gpu_lib.qrcp(Y, k, prec=prec)
    np.testing.assert_array_equal(piv.cpu().numpy(), piv_f.cpu().numpy())
    # downdated squared norms carry a few u of the initial ones: e^6 down at most, 2^-52 k e^6 relative
    np.testing.assert_allclose(rd.cpu().numpy(), rd_f.cpu().numpy(), rtol=1e-10)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_ties_go_to_the_lowest_column(gpu_lib, prec):
    """3000 columns of equal norm, more than the candidate set: 30 distinct unit directions, each repeated 100 times."""
    m, copies = 30, 100
    Y = torch.eye(m, dtype=torch.float64).repeat(copies, 1).cuda()
    piv, rd = gpu_lib.qrcp(Y, m, prec=prec)
    np.testing.assert_array_equal(piv.cpu().numpy(), np.arange(m))
    np.testing.assert_array_equal(rd.cpu().numpy(), np.ones(m))


def test_rank_deficient(gpu_lib):
    """Rank 5 and 20 steps: the steps past the rank pick distinct columns with residuals of rounding size."""
    rng = np.random.default_rng(3)
    Y = rng.standard_normal((2000, 5)) @ rng.standard_normal((5, 40))
    piv, rd = gpu_lib.qrcp(torch.from_numpy(Y), 20)
    piv, rd = piv.cpu().numpy(), rd.cpu().numpy()
    assert len(set(piv.tolist())) == 20
    assert np.all(rd[5:] <= 1e-6 * rd[0])   # sqrt of the rounding of downdated squared norms
