"""Values that are not finite in the triangular sweeps' right-hand side: they
reach exactly the rows that depend on them.  The matrix falls into two parts
that share every block of 256 rows (even and odd rows); entries of the even
part are poisoned with NaN, with the reserved payload of unwritten slots (in
FP64, and the value that FP32 narrows to its own) or with infinity.  The rows
that depend on a poisoned one, found on the host through the forward and then
the backward pattern, hold no finite value; all others are the oracle's.

Tolerances of the finite rows: those of the sweeps without such values."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1701_05913_amd as K  # noqa: E402
from tests.gpu_helpers import GpuSystem, pc_apply, relerr  # noqa: E402

NB = 1300
OFFSETS = {"rows": (2, 14, 260), "levels": (2, 14, 50, 64, 100, 260, 512)}
PAYLOADS = {"nan": np.uint64(0x7FF8000000000000), "f64_slot": np.uint64(0x7FFDEAD00BEEF001),
            "f32_slot": np.uint64(0x7FF81BD5A0000000), "inf": np.uint64(0x7FF0000000000000)}
PRECS = [(K.KRY_PREC_F64, "f64", 1e-12), (K.KRY_PREC_F32, "f32", 1e-5)]


def _system(bs, offsets):
    """Band of the given offsets, a third of the connections left out; no
    entry is zero."""
    rng = np.random.default_rng(bs)
    rows = [[i] for i in range(NB)]
    for d in offsets:
        for i in range(d, NB):
            if rng.random() < 0.67:
                rows[i].append(i - d)
                rows[i - d].append(i)
    rowptr = np.zeros(NB + 1, dtype=np.int32)
    rowptr[1:] = np.cumsum([len(r) for r in rows])
    col = np.concatenate([np.sort(r) for r in rows]).astype(np.int32)
    row = np.repeat(np.arange(NB), np.diff(rowptr))
    val = rng.uniform(0.5, 1.0, (col.size, bs, bs)) * rng.choice([-1.0, 1.0], (col.size, bs, bs))
    val *= 0.5 / (2 * len(offsets) * bs)
    val[col == row] += np.diag(1.0 + rng.random(bs))
    return dict(rowptr=rowptr, col=col, val=val.reshape(-1), bs=bs)


def _dependent(s, rows):
    """Rows whose result depends on the right-hand side of `rows`."""
    bad = np.zeros(NB, dtype=bool)
    bad[rows] = True
    for order, lower in ((range(NB), True), (range(NB - 1, -1, -1), False)):
        for i in order:
            c = s["col"][s["rowptr"][i]:s["rowptr"][i + 1]]
            bad[i] |= bad[c[c < i] if lower else c[c > i]].any()
    return bad


@pytest.mark.parametrize("prec,name,tol", PRECS)
@pytest.mark.parametrize("payload", list(PAYLOADS))
@pytest.mark.parametrize("bs", [1, 3])
@pytest.mark.parametrize("path", list(OFFSETS))
def test_reach(path, bs, payload, prec, name, tol):
    s = _system(bs, OFFSETS[path])
    A = oracle.Matrix.from_system(s)
    rows = np.array([520, 778])
    v = np.random.default_rng(4).standard_normal((NB, bs))
    clean = v.copy()
    v.view(np.uint64)[rows, bs - 1] = PAYLOADS[payload]
    bad = _dependent(s, rows)
    assert bad.any() and not bad[1::2].any()
    ref = oracle.PC(A, "bilu0", name).apply(clean.reshape(-1)).reshape(NB, bs)
    g = GpuSystem(s)
    try:
        z1, z2 = (z.reshape(NB, bs) for z in pc_apply(g, K.KRY_PC_ILU0, v.reshape(-1), prec=prec,
                                                      layout=K.KRY_SWEEP_LEVELS, repeat=2))
    finally:
        g.close()
    assert not np.isfinite(z1[bad]).any()
    if payload != "inf":
        assert np.isnan(z1[bad]).all()
    assert np.isfinite(z1[~bad]).all()
    assert relerr(z1[~bad], ref[~bad]) <= tol
    assert np.array_equal(z1, z2, equal_nan=True)
