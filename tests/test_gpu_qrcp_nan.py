"""Pivoted QR of a sketch with values that are not finite (they are not refused: a build's sketch may overflow): columns whose
norm is no number are never read as pivots while there are others, and a sketch of nothing else has no pivot."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


# up to and past the candidate set of 1024
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [1, 63, 300, 1024, 3000])
def test_no_number_at_all(gpu_lib, n, prec):
    Y = torch.full((n, 40), float("nan"), dtype=torch.float64, device="cuda")
    with pytest.raises(gpu_lib.KRRError) as e:
        gpu_lib.qrcp(Y, min(n, 20), prec=prec)
    assert e.value.status == -1


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n,good,k", [(200, 50, 70), (2000, 40, 90), (3000, 1500, 60)])
def test_some_columns(gpu_lib, n, good, k, prec):
    """The pivots are those of the finite columns alone, then distinct others."""
    l = 100
    rng = np.random.default_rng(n)
    Y = rng.standard_normal((n, l)) * np.exp(-2.0 * np.arange(l) / l) * (1 + rng.random((n, 1)))
    bad = np.sort(rng.permutation(n)[good:])
    Y[bad, rng.integers(0, l, len(bad))] = np.nan
    piv = gpu_lib.qrcp(torch.from_numpy(Y), k, prec=prec)[0].cpu().numpy()
    fine = np.setdiff1d(np.arange(n), bad)
    m = min(good, k)
    alone = gpu_lib.qrcp(torch.from_numpy(Y[fine]), m, prec=prec)[0].cpu().numpy()
    np.testing.assert_array_equal(piv[:m], fine[alone])
    assert len(set(piv.tolist())) == k and piv.min() >= 0 and piv.max() < n
