"""An entry of the launch table that was tuned among staged forms does not take a product of few FP64 pairs off its path."""
import json

import numpy as np
import pytest
import torch

from test_launch_record import lib  # noqa: F401  (fixture)


@pytest.fixture
def table(lib, tmp_path):  # noqa: F811
    """A table with an entry for FP64, d = 3, 1024 to 2047 points, square; forgotten afterwards."""
    f = tmp_path / "table.json"
    f.write_text(json.dumps({"arch": "", "entries": {"0:3:1:10:1": [0, 0]}}))
    lib.autotune_load(str(f))
    yield
    lib.set_variant(3, 1, "fp64", -1)


def test_variant_with_a_tuned_entry(lib, table):  # noqa: F811
    assert lib.kmv_variant(3, 1, "fp64", square=True, n=1500) == (-1, False)
    lib.set_variant(3, 1, "fp64", 2)   # a forced one is run
    assert lib.kmv_variant(3, 1, "fp64", square=True, n=1500) == (2, False)


@pytest.mark.gpu
def test_product_with_a_tuned_entry(gpu_lib, table):
    X = torch.from_numpy(np.random.default_rng(0).random((1500, 3)))
    v = torch.from_numpy(np.random.default_rng(1).standard_normal(1500))
    with_entry = gpu_lib.kernel_mv(X, None, 0.1, v, prec="fp64")
    assert gpu_lib.kmv_last_launch()[0] == -1
    gpu_lib.set_variant(3, 1, "fp64", 0)
    forced = gpu_lib.kernel_mv(X, None, 0.1, v, prec="fp64")
    assert gpu_lib.kmv_last_launch()[0] == 0
    gpu_lib.set_variant(3, 1, "fp64", -1)
    assert torch.equal(with_entry, gpu_lib.kernel_mv(X, None, 0.1, v, prec="fp64"))
    torch.testing.assert_close(with_entry, forced, rtol=0, atol=2.0 ** -52 * 100 * float(v.abs().sum()))
