"""Products of few FP64 pairs straight from the caller's arrays, at the edges of their target tiles (2, 8 and 32 targets:
up to 1024, 4096 and more rows), source splits and column counts; staging with few targets; and the scan of the inputs."""
import numpy as np
import pytest
import torch

from oracle import kernel as ok

pytestmark = pytest.mark.gpu


def _check(gpu_lib, m, n, d, R, deriv, prec="fp64", same=False, shift=None, seed=0):
    rng = np.random.default_rng(seed + 131 * m + n)
    Y = rng.random((n, d))
    X = Y if same else rng.random((m, d))
    V = rng.standard_normal((n, R))
    eps = 0.3 * d
    U = gpu_lib.kernel_mv(torch.from_numpy(X), None if same else torch.from_numpy(Y), eps, torch.from_numpy(V),
                          shift=shift, deriv=deriv, prec=prec).cpu().numpy()
    K = ok.kernel_mv(X, Y, eps, V)
    if shift is not None:
        K = K + np.asarray(shift) * V
    Kd = ok.kernel_mv(X, Y, eps, V, deriv=1) if deriv else None
    ref = K if deriv == 0 else Kd if deriv == 1 else np.hstack([K, Kd])
    # every weight is at most 1 and off by at most 100 roundings; sums of n (FP32: up to n) terms add as many
    u = 2.0 ** -52 if prec == "fp64" else 2.0 ** -23
    tol = u * (n + 100) * np.abs(V).sum(axis=0).max() + 1e-13
    assert np.abs(U.reshape(ref.shape) - ref).max() <= tol


@pytest.mark.parametrize("m,n,d,R,deriv", [
    (1, 1, 1, 1, 0), (2, 3, 3, 1, 1), (3, 7, 2, 1, 2), (1, 70001, 5, 1, 0), (5, 33333, 8, 3, 0), (16, 8193, 8, 1, 2),
    (1024, 2049, 4, 1, 0), (1025, 2047, 7, 5, 0), (1023, 8191, 3, 1, 2), (4096, 2048, 16, 8, 0), (4097, 500, 13, 4, 0),
    (200001, 31, 3, 1, 1), (4095, 255, 6, 2, 0)])
def test_matches_oracle(gpu_lib, m, n, d, R, deriv):
    _check(gpu_lib, m, n, d, R, deriv)


@pytest.mark.parametrize("n,d,R,shift", [(1, 2, 1, 0.5), (777, 3, 1, 1e-3), (2896, 8, 1, 0.25), (2897, 8, 1, 0.25),
                                         (1500, 5, 3, [0.0, 1.0, 2.0])])
def test_same_points_with_ridge(gpu_lib, n, d, R, shift):
    _check(gpu_lib, n, n, d, R, 0, same=True, shift=shift)


# staged: few targets (padded less than the sources), more FP64 pairs than the direct kernel takes
@pytest.mark.parametrize("prec", ["fp64", "fp32", "mixed"])
@pytest.mark.parametrize("m,n,d,R", [(1, 5000, 3, 1), (63, 9001, 8, 1), (65, 4097, 17, 1), (130, 70001, 3, 3), (257, 3001, 5, 9)])
def test_few_targets(gpu_lib, prec, m, n, d, R):
    _check(gpu_lib, m, n, d, R, 0, prec=prec)


@pytest.mark.parametrize("n", [3000, 6001, 12289])
def test_same_points_small_symmetric(gpu_lib, n):
    _check(gpu_lib, n, n, 6, 1, 0, same=True, shift=0.1)


def test_result_over_its_input(gpu_lib):
    """U in V's own memory: accepted at every size."""
    rng = np.random.default_rng(5)
    X, v = rng.random((300, 3)), rng.standard_normal(300)
    Xd, vd = torch.from_numpy(X).cuda(), torch.from_numpy(v).cuda()
    lib = gpu_lib.load()
    assert lib.krr_kernel_mv(Xd.data_ptr(), 300, Xd.data_ptr(), 300, 3, 0.5, vd.data_ptr(), 1, None, 0, 0, vd.data_ptr(), 0) == 0
    np.testing.assert_allclose(vd.cpu().numpy(), ok.kernel_mv(X, X, 0.5, v), rtol=0, atol=2.0 ** -52 * 400 * np.abs(v).sum())


@pytest.mark.parametrize("n", [1, 129, 4001])
@pytest.mark.parametrize("at", ["first", "last"])
@pytest.mark.parametrize("prec,d", [("fp64", 3), ("fp64", 31), ("mixed", 128)])
def test_scan_finds_one_bad_value(gpu_lib, n, at, prec, d):
    """In the first and the last value of each input, whatever the chunk it falls in; the result is left unwritten."""
    rng = np.random.default_rng(n + d)
    good = {"Xt": rng.random((n + 2, d)), "Xs": rng.random((n, d)), "V": rng.standard_normal((n, 1))}
    lib = gpu_lib.load()
    for name in good:
        args = {k: torch.from_numpy(v.copy()).cuda() for k, v in good.items()}
        args[name].view(-1)[0 if at == "first" else -1] = float("-inf")
        U = torch.full((n + 2, 1), 7.0, dtype=torch.float64, device="cuda")
        rc = lib.krr_kernel_mv(args["Xt"].data_ptr(), n + 2, args["Xs"].data_ptr(), n, d, 1.0, args["V"].data_ptr(), 1,
                               None, 0, 0 if prec == "fp64" else 2, U.data_ptr(), 0)
        assert rc == -1 and name.encode() in lib.krr_last_error()
        assert bool((U == 7.0).all())


# mixed, same points: super-tiles of 1024 shared by four blocks, whole and cut off at every part (512 points, 64 padding)
@pytest.mark.parametrize("n", [1, 511, 513, 1025, 3071, 3073, 9217])
@pytest.mark.parametrize("d", [2, 9, 16])
def test_same_points_mixed_parts(gpu_lib, n, d):
    _check(gpu_lib, n, n, d, 1, 0, prec="mixed", same=True, shift=0.1)


# many 32-bit columns without a block kernel: derivatives, and more than 20 coordinates
@pytest.mark.parametrize("prec", ["fp32", "mixed"])
@pytest.mark.parametrize("n,d,R,deriv", [(918, 54, 64, 0), (300, 33, 9, 0), (1100, 6, 33, 2), (257, 3, 9, 1), (130, 20, 40, 2)])
def test_many_columns_without_a_block_kernel(gpu_lib, prec, n, d, R, deriv):
    _check(gpu_lib, n, n, d, R, deriv, prec=prec, same=True)


# the direct forms' coordinate and column counts: every d up to 32 at its staged width, chunks of one to eight columns
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("d,R,deriv", [(1, 3, 0), (5, 7, 0), (7, 6, 0), (9, 1, 2), (10, 2, 0), (11, 4, 0), (12, 5, 0), (13, 8, 0),
                                       (15, 7, 0), (17, 1, 0), (20, 3, 0), (21, 1, 2), (26, 6, 0), (27, 1, 0), (32, 7, 0)])
def test_direct_counts(gpu_lib, prec, d, R, deriv):
    _check(gpu_lib, 2100, 4200, d, R, deriv, prec=prec)


# FP64, 33 to 128 coordinates: sixteens of coordinates, one target to several tiles, column chunks, both kernels
@pytest.mark.parametrize("m,n,d,R,deriv", [(1, 1, 33, 1, 0), (20, 511, 90, 1, 0), (65, 257, 48, 1, 2), (300, 1000, 64, 4, 0),
                                           (64, 5000, 65, 9, 2), (1000, 70, 128, 3, 0), (257, 256, 49, 1, 1)])
def test_many_coordinates(gpu_lib, m, n, d, R, deriv):
    _check(gpu_lib, m, n, d, R, deriv)
