"""Kernel products held to their own rounding, at every edge of the paths that few pairs, few targets, shared super-tiles,
32-bit columns without a block kernel and reduced coordinate counts take.

A weight is off by at most some tens of roundings (its squared distance, 3.3 eps at most here, and its exponential), and V's
signs are random, so a sum's error is that many roundings of sigma_i = (sum_j (K_ij V_j)^2)^(1/2), six times over for the
largest of up to 10^5 entries, and the sums of up to 512 32-bit terms between their FP64 folds add some tens more: 512 units
of 2^-24 sigma_i, and 1024 of 2^-53 in FP64 (whose sums are longer).  Leaving out a coordinate or 512 sources moves an
entry by a large part of sigma_i, thousands of times more."""
import numpy as np
import pytest
import torch

from oracle import kernel as ok

UNITS = {"fp64": 1024 * 2.0 ** -53, "fp32": 512 * 2.0 ** -24, "mixed": 512 * 2.0 ** -24}

FEW_TARGETS = [(1, 5000, 3, 1), (63, 9001, 8, 1), (65, 4097, 17, 1), (130, 70001, 3, 3), (257, 3001, 5, 9)]
# super-tiles of 1024 shared by four blocks, whole and cut off at every part
PARTS = [(n, d) for n in (513, 1025, 3071, 3073, 9217) for d in (2, 9, 16)]
NO_BLOCK = [(918, 54, 64, 0), (300, 33, 9, 0), (1100, 6, 33, 2), (257, 3, 9, 1), (130, 20, 40, 2)]
COUNTS = [(1, 3, 0), (5, 7, 0), (7, 6, 0), (9, 1, 2), (10, 2, 0), (11, 4, 0), (12, 5, 0), (13, 8, 0), (15, 7, 0), (17, 1, 0),
          (20, 3, 0), (21, 1, 2), (26, 6, 0), (27, 1, 0), (32, 7, 0), (54, 1, 0), (90, 3, 0)]
# few pairs: one target to a thread up to 512, four groups to a block up to 512 sources, one split up to 64 pairs a thread
EDGES = [(m, n, d, R, deriv) for m in (511, 512, 513) for n in (511, 512, 513)
         for d, R, deriv in ((3, 1, 0), (3, 4, 0), (3, 1, 1), (16, 8, 0), (16, 1, 2))]
SPLITS = [(600, 2048, 3, 1, 0), (600, 2049, 3, 1, 0), (600, 4096, 3, 4, 0), (600, 4097, 3, 4, 0), (20, 16384, 3, 1, 2),
          (20, 16385, 3, 1, 2), (60, 16384, 16, 1, 0), (60, 16385, 16, 1, 0)]


def problem(m, n, d, R, same=False):
    rng = np.random.default_rng(131 * m + n)
    Y = rng.random((n, d))
    return (Y if same else rng.random((m, d))), Y, rng.standard_normal((n, R)), 0.3 * d


def reference(X, Y, V, eps, deriv):
    K = ok.kernel_mv(X, Y, eps, V)
    sigma = np.sqrt(ok.kernel_mv(X, Y, eps / 2, V ** 2))   # K^2 is the kernel of eps / 2
    if deriv == 0:
        return K, sigma
    Kd = ok.kernel_mv(X, Y, eps, V, deriv=1)               # (D^2 / eps) K, D^2 / eps <= 1 / 0.3, off by K's share too
    sd = (1 + 1 / 0.3) * sigma
    return (Kd, sd) if deriv == 1 else (np.hstack([K, Kd]), np.hstack([sigma, sd]))


def check(gpu_lib, m, n, d, R, deriv, prec, same=False):
    X, Y, V, eps = problem(m, n, d, R, same)
    U = gpu_lib.kernel_mv(torch.from_numpy(X), None if same else torch.from_numpy(Y), eps, torch.from_numpy(V), deriv=deriv,
                          prec=prec).cpu().numpy()
    ref, sigma = reference(X, Y, V, eps, deriv)
    worst = np.abs((U.reshape(ref.shape) - ref) / sigma).max()
    assert worst <= UNITS[prec], worst / UNITS[prec]


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp64", "fp32", "mixed"])
@pytest.mark.parametrize("m,n,d,R", FEW_TARGETS)
def test_few_targets(gpu_lib, prec, m, n, d, R):
    check(gpu_lib, m, n, d, R, 0, prec)


@pytest.mark.gpu
@pytest.mark.parametrize("n,d", PARTS)
def test_same_points_mixed_parts(gpu_lib, n, d):
    check(gpu_lib, n, n, d, 1, 0, "mixed", same=True)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [3000, 6001, 12289])
def test_same_points_small_symmetric(gpu_lib, n):
    check(gpu_lib, n, n, 6, 1, 0, "fp64", same=True)


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp32", "mixed"])
@pytest.mark.parametrize("n,d,R,deriv", NO_BLOCK)
def test_many_columns_without_a_block_kernel(gpu_lib, prec, n, d, R, deriv):
    check(gpu_lib, n, n, d, R, deriv, prec, same=True)


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("d,R,deriv", COUNTS)
def test_coordinate_counts(gpu_lib, prec, d, R, deriv):
    check(gpu_lib, 2100, 4200, d, R, deriv, prec)


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,d,R,deriv", EDGES + SPLITS)
def test_few_pairs(gpu_lib, m, n, d, R, deriv):
    check(gpu_lib, m, n, d, R, deriv, "fp64")
    if R == 1 or deriv == 0:
        assert gpu_lib.kmv_last_launch()[0] == -1   # straight from the arrays


@pytest.mark.parametrize("m,n,d,R,deriv", [(63, 9001, 8, 1, 0), (918, 918, 54, 64, 0),
                                           (2100, 4200, 32, 7, 0), (1025, 1025, 16, 1, 0), (511, 513, 16, 1, 2)])
def test_bound_sees_what_is_left_out(m, n, d, R, deriv):
    """The same bound against references that leave out the last coordinate, or 512 of the sources."""
    X, Y, V, eps = problem(m, n, d, R, same=m == n)
    ref, sigma = reference(X, Y, V, eps, deriv)
    dropped, _ = reference(X[:, :-1], Y[:, :-1], V, eps, deriv)
    Vs = V.copy()
    Vs[-512:] = 0.0
    fewer, _ = reference(X, Y, Vs, eps, deriv)
    for wrong in (dropped, fewer):
        assert np.abs((wrong - ref) / sigma).max() > 100 * UNITS["fp32"]
