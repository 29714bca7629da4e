"""Dot products that return to the host, from more threads at once than there
are workspace slots for them: every call gets its own result.

Tolerance: one sum of products in double over at most 700 001 terms against
numpy's: 1e-12 of the sum of magnitudes."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1701_05913_amd as K  # noqa: E402


def test_many_threads():
    sizes = [1, 255, 256, 257, 2880, 131072, 131073, 700001, 5, 64, 4097, 99999]
    jobs = []
    for i, n in enumerate(sizes):
        rng = np.random.default_rng(i)
        x, y = rng.standard_normal(n), rng.standard_normal(n)
        m = K.MapCreateLocal(n)
        xt, yt = torch.from_numpy(x).to("cuda:0"), torch.from_numpy(y).to("cuda:0")
        jobs.append((m, K.VecWrap(m, xt), K.VecWrap(m, yt), float(x @ y), float(np.abs(x * y).sum()), xt, yt))
    torch.cuda.synchronize()
    bad = []

    def work(j):
        for _ in range(20):
            d = K.VecDot(j[1], j[2])
            if not abs(d - j[3]) <= 1e-12 * j[4]:
                bad.append((d, j[3]))

    threads = [threading.Thread(target=work, args=(j,)) for j in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for j in jobs:
        K.VecDestroy(j[1])
        K.VecDestroy(j[2])
        K.MapDestroy(j[0])
    assert not bad
