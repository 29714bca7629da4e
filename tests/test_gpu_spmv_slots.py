"""Sparse product over slices of every width from 0 to 11 slots (whole batches
and every remainder), rows shorter than their slice (padding), a last slice
that is not full, infinities beside padding, against a plain sum.

Tolerance: each row sums at most 33 products in double: 1e-14 of the largest
row sum."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1701_05913_amd as K  # noqa: E402
from tests.gpu_helpers import GpuSystem  # noqa: E402


@pytest.mark.parametrize("bs", [1, 3])
@pytest.mark.parametrize("width", range(1, 12))
def test_widths(width, bs):
    rng = np.random.default_rng(width)
    nb = 64 * 4 + 17
    rowptr, col = [0], []
    for i in range(nb):
        w = width if i % 64 == 5 else int(rng.integers(1, width + 1))
        c = set(rng.choice(nb - 1, size=w - 1, replace=False) + 1 if w > 1 else [])
        c.add(i)
        col += sorted(int(q) for q in c)
        rowptr.append(len(col))
    val = rng.standard_normal((len(col), bs, bs))
    x = rng.standard_normal((nb, bs))
    x[0] = np.inf                        # only row 0 reads it; padding must not
    s = dict(rowptr=np.array(rowptr, np.int32), col=np.array(col, np.int32), val=val.reshape(-1), bs=bs)
    ref = np.zeros((nb, bs))
    big = np.zeros((nb, bs))
    row = np.repeat(np.arange(nb), np.diff(rowptr))
    with np.errstate(invalid="ignore"):
        t = np.einsum("prc,pc->pr", val, x[col])
        np.add.at(ref, row, t)
        np.add.at(big, row, np.abs(val).sum(2) * 4.0)
    g = GpuSystem(s)
    try:
        xt, xh = g.vec(x.reshape(-1))
        yt, yh = g.vec()
        K.MatVecMXY(g.A, xh, yh)
        torch.cuda.synchronize()
        y = yt.cpu().numpy().reshape(nb, bs)
    finally:
        g.close()
    assert np.all(np.isfinite(y[1:]))
    assert np.max(np.abs(y[1:] - ref[1:]) / big[1:]) <= 1e-14
