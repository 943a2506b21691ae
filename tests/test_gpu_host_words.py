"""The pinned words that the scan and the pivoted QR hand their results back in: kept for the process, shared by its threads
and streams, not allocated for every thread."""
import threading

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _mappings():
    with open("/proc/self/maps") as f:
        return sum(1 for _ in f)


def _one_after_another(work, count):
    for _ in range(count):
        t = threading.Thread(target=work)
        t.start()
        t.join()


@pytest.mark.parametrize("what", ["qr", "scan"])
def test_threads_that_end(gpu_lib, what):
    """64 threads, each gone before the next: every pinned allocation is a mapping of its own."""
    Y = torch.rand(200, 30, dtype=torch.float64, device="cuda")

    def work():
        if what == "qr":
            gpu_lib.qrcp(Y, 20)
        else:
            gpu_lib.kernel_mv(Y, None, 5.0, Y[:, 0], prec="mixed")

    _one_after_another(work, 4)
    before = _mappings()
    _one_after_another(work, 64)
    assert _mappings() - before < 32


def test_threads_and_streams_together(gpu_lib):
    """Eight threads with a stream each: every result is its own input's, and a bad value is reported to its own call."""
    rng = np.random.default_rng(1)
    X = [torch.from_numpy(rng.random((n, 3))).cuda() for n in (90, 400, 2500, 7000, 90, 400, 2500, 7000)]
    Y = [torch.from_numpy(rng.standard_normal((1500 + 100 * i, 40))).cuda() for i in range(8)]
    bad = [x.clone() for x in X]
    for b in bad:
        b[-1, 1] = float("nan")
    alone = [(gpu_lib.kernel_mv(x, None, 0.2, x[:, 0]), gpu_lib.qrcp(y, 33)) for x, y in zip(X, Y)]
    torch.cuda.synchronize()
    wrong = []

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for rep in range(10):
                U = gpu_lib.kernel_mv(X[i], None, 0.2, X[i][:, 0])
                piv, rd = gpu_lib.qrcp(Y[i], 33)
                torch.cuda.current_stream().synchronize()
                if not (torch.equal(U, alone[i][0]) and torch.equal(piv, alone[i][1][0]) and torch.equal(rd, alone[i][1][1])):
                    wrong.append((i, rep))
                try:
                    gpu_lib.kernel_mv(bad[i], None, 0.2, X[i][:, 0])
                    wrong.append((i, rep, "accepted"))
                except gpu_lib.KRRError as e:
                    if e.status != -1:
                        wrong.append((i, rep, e.status))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(8)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
