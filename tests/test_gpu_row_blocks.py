"""Triangular sweeps over row blocks (general patterns, no grid stencil) at the
sizes where they can go wrong: one row, a wavefront, a block of 256 rows, one
row less and more, several blocks; three and six dependencies a row (the two
widths of the kernel) and seven (the level sweeps); rows that read the row
before (chains inside a wavefront) and rows of earlier blocks, rows without
dependencies.

Tolerances: the blocks are diagonally dominant (row sums of the off-diagonal
part at most half the diagonal), so that errors don't grow along a chain: the
FP64 apply differs from the oracle by a few ulps a row, far below 1e-12.
FP32 factors: a few FP32 ulps (6e-8), below 1e-5.  BF16 factors may fall on
the other side of a rounding boundary (2^-8 of an entry): 1e-4."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1701_05913_amd as K  # noqa: E402
from tests.gpu_helpers import GpuSystem, pc_apply, relerr  # noqa: E402

PRECS = [(K.KRY_PREC_F64, "f64", 1e-12), (K.KRY_PREC_F32, "f32", 1e-5),
         (K.KRY_PREC_BF16_FACTORS, "bf16", 1e-4)]
OFFSETS = {3: (1, 7, 130), 6: (1, 2, 9, 64, 255, 300), 7: (1, 2, 9, 64, 255, 300, 513)}


def _system(nb, bs, offsets, seed):
    """Band of the given offsets, a fifth of the connections left out."""
    rng = np.random.default_rng(seed)
    rows = [[i] for i in range(nb)]
    for d in offsets:
        for i in range(d, nb):
            if rng.random() < 0.8:
                rows[i].append(i - d)
                rows[i - d].append(i)
    rowptr = np.zeros(nb + 1, dtype=np.int32)
    rowptr[1:] = np.cumsum([len(r) for r in rows])
    col = np.concatenate([np.sort(r) for r in rows]).astype(np.int32)
    row = np.repeat(np.arange(nb), np.diff(rowptr))
    val = rng.uniform(-1.0, 1.0, (col.size, bs, bs)) * (0.5 / (2 * len(offsets) * bs))
    val[col == row] += np.diag(1.0 + rng.random(bs))
    return dict(rowptr=rowptr, col=col, val=val.reshape(-1), bs=bs)


@pytest.mark.parametrize("prec,name,tol", PRECS)
@pytest.mark.parametrize("bs", [1, 3])
@pytest.mark.parametrize("width", [3, 6, 7])
@pytest.mark.parametrize("nb", [1, 64, 255, 256, 257, 2600])
def test_general_pattern_sweeps(nb, width, bs, prec, name, tol):
    s = _system(nb, bs, OFFSETS[width], seed=nb + width)
    A = oracle.Matrix.from_system(s)
    v = np.random.default_rng(4).standard_normal(A.n)
    ref = oracle.PC(A, "bilu0", name).apply(v)
    g = GpuSystem(s)
    try:
        z1, z2 = pc_apply(g, K.KRY_PC_ILU0, v, prec=prec, layout=K.KRY_SWEEP_LEVELS, repeat=2)
    finally:
        g.close()
    assert relerr(z1, ref) <= tol
    assert np.array_equal(z1, z2)


def test_not_a_number_does_not_stall():
    """NaNs in the right-hand side, the reserved payload of unwritten slots
    among them, come out as NaNs in every row that depends on them."""
    s = _system(600, 3, OFFSETS[3], seed=2)
    v = np.random.default_rng(4).standard_normal(1800)
    v.view(np.uint64)[[0, 5]] = 0x7FFDEAD00BEEF001
    v[7] = np.inf
    g = GpuSystem(s)
    try:
        z1, z2 = pc_apply(g, K.KRY_PC_ILU0, v, layout=K.KRY_SWEEP_LEVELS, repeat=2)
    finally:
        g.close()
    assert np.isnan(z1[:9]).any()
    assert np.array_equal(np.isnan(z1), np.isnan(z2))
