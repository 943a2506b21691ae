"""What the library says about its launches (krr_kmv_variant, krr_kmv_last_launch, krr_cull_stats) where FP64 products of few
pairs run outside the launch table, and for targets staged in fewer than 1024 rows."""
import os

import pytest
import torch


@pytest.fixture
def lib():
    import paper_1905_10587_amd as krr
    if not os.path.exists(krr.library_path()):
        from paper_1905_10587_amd import build
        build.build()
    return krr


def _pairs(d, R):
    return (1 << 23) >> ((3 if d > 8 else 0) + (1 if R > 1 else 0))


@pytest.mark.parametrize("d,R,deriv", [(3, 1, 0), (8, 1, 2), (9, 1, 0), (16, 8, 0), (2, 2, 0)])
def test_variant_of_few_pairs(lib, d, R, deriv):
    n = int(_pairs(d, R) ** 0.5)   # the largest square product
    assert lib.kmv_variant(d, R, "fp64", deriv=deriv, square=True, n=n) == (-1, False)
    assert lib.kmv_variant(d, R, "fp64", deriv=deriv, square=True, n=n + 1)[0] >= 0
    assert lib.kmv_variant(d, R, "fp64", deriv=deriv, square=True)[0] >= 0       # size unknown
    assert lib.kmv_variant(d, R, "fp64", deriv=deriv, square=False, n=n)[0] >= 0
    assert lib.kmv_variant(d, R, "mixed", deriv=deriv, square=True, n=n)[0] >= 0
    lib.set_variant(d, R, "fp64", 1)   # a forced variant is what runs
    try:
        assert lib.kmv_variant(d, R, "fp64", deriv=deriv, square=True, n=n) == (1, False)
    finally:
        lib.set_variant(d, R, "fp64", -1)
    assert lib.kmv_variant(17, 1, "fp64", square=True, n=100)[0] >= 0
    assert lib.kmv_variant(3, 2, "fp64", deriv=1, square=True, n=100)[0] >= 0


@pytest.mark.gpu
def test_record_after_few_pairs(gpu_lib):
    X = torch.rand(9000, 8, dtype=torch.float64, device="cuda")
    v = torch.rand(9000, dtype=torch.float64, device="cuda")
    gpu_lib.kernel_mv(X, None, 0.3, v, prec="mixed")
    assert gpu_lib.kmv_last_launch()[0] >= 0 and gpu_lib.cull_stats()[0] == 9216 ** 2
    S = X[:600].contiguous()
    gpu_lib.kernel_mv(S, None, 0.3, v[:600], prec="fp64")
    variant, split, sym = gpu_lib.kmv_last_launch()
    assert (variant, sym) == (-1, False) and 0 < split <= 600
    assert gpu_lib.cull_stats() == (1024 ** 2, 0)


@pytest.mark.gpu
def test_record_after_a_culled_product(gpu_lib):
    """The culled product's skipped pairs are not those of the product after it."""
    X = 200.0 * torch.rand(9000, 3, dtype=torch.float64, device="cuda")
    v = torch.rand(9000, dtype=torch.float64, device="cuda")
    gpu_lib.set_cull(1)
    try:
        gpu_lib.kernel_mv(X, None, 0.3, v, prec="mixed")
        assert gpu_lib.cull_stats()[1] > 0
        gpu_lib.kernel_mv(X[:100].contiguous(), X, 0.3, v, prec="fp64")
        assert gpu_lib.cull_stats() == (1024 ** 2, 0)
    finally:
        gpu_lib.set_cull(-1)


@pytest.mark.gpu
@pytest.mark.parametrize("prec,m", [("mixed", 70), ("fp64", 300), ("fp32", 1025)])
def test_total_of_few_targets(gpu_lib, prec, m):
    X = torch.rand(70000, 3, dtype=torch.float64, device="cuda")
    gpu_lib.kernel_mv(X[:m].contiguous(), X, 0.3, X[:, 0], prec=prec)
    assert gpu_lib.kmv_last_launch()[0] >= 0
    assert gpu_lib.cull_stats()[0] == (-(-m // 1024) * 1024) ** 2
