"""krr_init loads the block apply's kernels: the first apply to several columns of a process takes no device memory."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# the allocator is given what the applies need first, so that memory that goes is a code object's
SCRIPT = """
import sys
import torch
blocks = [torch.empty(1 << 20, dtype=torch.uint8, device="cuda") for _ in range(64)]
del blocks
import paper_1905_10587_amd as krr
prec = sys.argv[1]
X = torch.rand(600, 3, dtype=torch.float64, device="cuda")
P = krr.Preconditioner(X, 0.05, [1e-3], 70, anchors=torch.arange(70), prec=prec)
x = torch.rand(600, 4, dtype=torch.float64, device="cuda")
P.apply(x[:, 0])
torch.cuda.synchronize()
before = torch.cuda.mem_get_info()[0]
P.apply(x)
torch.cuda.synchronize()
print("taken", before - torch.cuda.mem_get_info()[0])
"""


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_first_block_apply(gpu_lib, prec):
    r = subprocess.run([sys.executable, "-c", SCRIPT, prec], cwd=ROOT, capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
    assert "taken 0" in r.stdout.splitlines()
