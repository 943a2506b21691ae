"""Calls whose launches would hold 2^32 threads or more along one dimension of a grid: such a launch runs cut short without
an error, so its kernels number their blocks over two dimensions."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def room(gpu_lib):
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs 80 GB of device memory")
    yield
    torch.cuda.empty_cache()


def _rand(*shape, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)


def test_staged_values(gpu_lib):
    """32 million sources of 65 coordinates (staged as 128) and four columns: 4.35e9 staged values in one launch."""
    n, d, eps = 32_000_000, 65, 10.0
    X, V = _rand(n, d, seed=1), _rand(n, 4, seed=2)
    T = X[-3:].contiguous()
    U = gpu_lib.kernel_mv(T, X, eps, V, prec="fp32")
    ref = torch.zeros(3, 4, dtype=torch.float64, device="cuda")
    for i in range(0, n, 4_000_000):
        for a in range(3):
            ref[a] += torch.exp(-((X[i:i + 4_000_000] - T[a]) ** 2).sum(1) / eps) @ V[i:i + 4_000_000]
    # positive terms: the weights' 32-bit errors (some tens of 2^-24 each) stay relative
    torch.testing.assert_close(U, ref, rtol=1e-5, atol=0)


def test_finished_rows(gpu_lib):
    """1.08e9 targets of one column: four threads to a row of the finishing pass."""
    m, n, eps = 1_080_000_000, 8, 0.3
    T, S, v = _rand(m, 1, seed=3), _rand(n, 1, seed=4), _rand(n, seed=5)
    U = gpu_lib.kernel_mv(T, S, eps, v, prec="fp32")
    for rows in (slice(0, 4096), slice(m // 2, m // 2 + 4096), slice(m - 4096, m)):
        ref = torch.exp(-(T[rows] - S.T) ** 2 / eps) @ v
        torch.testing.assert_close(U[rows], ref, rtol=1e-5, atol=0)


def test_applied_rows(gpu_lib):
    """5.4e8 rows, two columns: eight threads to a row of the pass W Z; each column as by itself."""
    n, eps, k = 540_000_000, 0.3, 2
    X = _rand(n, 1, seed=6)
    P = gpu_lib.Preconditioner(X, eps, [0.5], k, anchors=torch.tensor([0, n - 1]), prec="fp64")
    del X
    x = _rand(n, 2, seed=7)
    out = P.apply(x)
    for c in range(2):
        one = P.apply(x[:, c].contiguous())
        # sums over n rows in two orders: a relative difference of a few n^(1/2) 2^-53 of W z, which is below x
        assert bool(((out[:, c] - one).abs().max() <= 1e-9))
        del one
