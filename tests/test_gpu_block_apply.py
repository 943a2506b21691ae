"""The preconditioner's apply to 2 .. 256 columns at the edges of its tiles (16, 32 and 64 of the columns, 64 columns of W,
16 and 32 rows, fewer than four columns or rows, row splits), and to more, against one column at a time."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n,k,R", [(5, 1, 2), (16, 3, 3), (17, 16, 16), (19, 5, 4), (300, 63, 5), (1024, 64, 16), (1025, 65, 15),
                                   (3000, 131, 4), (20001, 259, 8), (300, 70, 33), (130, 20, 100), (90, 33, 257),
                                   (16400, 66, 64)])
def test_block_equals_columns(gpu_lib, n, k, R, prec):
    rng = np.random.default_rng(n + k)
    X = torch.from_numpy(rng.random((n, 6))).cuda()
    betas = [0.5, 2.0, 8.0]
    P = gpu_lib.Preconditioner(X, 0.4, betas, k, anchors="fps", prec=prec)
    V = torch.from_numpy(rng.standard_normal((n, R))).cuda()
    bs = [betas[(r * r) % 3] for r in range(R)]
    out = P.apply(V, bs, prec=prec)
    ref = torch.stack([P.apply(V[:, r].contiguous(), [bs[r]], prec=prec) for r in range(R)], dim=1)
    # z = G t: sums of n and of k terms in another order; |W^T x| <= |W| |x|, |G| <= 1 / beta, and |W|^2 <= |K| <= n
    err = (out - ref).abs().max().item()
    assert err <= 2.0 ** -52 * 4 * (n + 2 * k) * (1 + n / 0.5) / 0.5 * V.abs().max().item()
    # the same columns again beside them, up to the next tile and past it
    wide = P.apply(torch.cat([V] * (16 // R + 1), dim=1).contiguous(), bs * (16 // R + 1), prec=prec)
    assert (wide[:, :R] - out).abs().max().item() <= 2.0 ** -52 * 4 * (n + 2 * k) * (1 + n / 0.5) / 0.5 * V.abs().max().item()
