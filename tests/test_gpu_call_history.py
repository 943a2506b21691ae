"""A product's split of its sources, and so its bits, do not depend on the products that the process ran before it."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SCRIPT = """
import hashlib, sys
import torch
import paper_1905_10587_amd as krr
prec, n, d, before, R = sys.argv[1], int(sys.argv[2]), int(sys.argv[3]), int(sys.argv[4]), int(sys.argv[5])
g = torch.Generator(device="cuda").manual_seed(1)
X = torch.rand(n, d, generator=g, device="cuda", dtype=torch.float64)
V = torch.randn(n, 128, generator=g, device="cuda", dtype=torch.float64)
if before:
    krr.kernel_mv(X, None, 0.3, V[:, :before].contiguous(), prec=prec)
U = krr.kernel_mv(X, None, 0.3, V[:, :R].contiguous(), prec=prec)
print("result", krr.kmv_last_launch(), hashlib.sha256(U.cpu().numpy().tobytes()).hexdigest())
"""


def _run(*args):
    r = subprocess.run([sys.executable, "-c", SCRIPT, *map(str, args)], cwd=ROOT, capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
    return [line for line in r.stdout.splitlines() if line.startswith("result")]


# FP64 matrix cores (column groups of a block), FP64 direct (chunks of 4 and 8), staged V (column tiles), per-wave block form
@pytest.mark.parametrize("prec,before,R", [("fp64", 16, 128), ("fp64", 4, 8), ("mixed", 128, 40), ("mixed", 16, 32)])
def test_fresh_process_and_after_other_columns(gpu_lib, prec, before, R):
    assert _run(prec, 20000, 6, before, R) == _run(prec, 20000, 6, 0, R)
