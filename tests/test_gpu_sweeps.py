"""Grid-tiled triangular sweeps at the edges of their tiling, against the
oracle: tiles narrower than 8 lines (every TJ from 2 to 7, with TK up to 32),
ragged last tiles, lines and step counts around the result ring's and the
right-hand side ring's lengths, and several tiles per workgroup queue.

Tolerances: the FP64 apply differs from the oracle by rounding order alone;
both solve the same triangular systems, whose error is a few ulps times the
number of hyperplanes, so 1e-12 is far above it and far below any wrong
value.  FP32 factors are compared with the oracle's emulation of the same
rounding, which sums in another order: a few FP32 ulps (6e-8) per hyperplane
over at most 150 hyperplanes stays below 1e-5.  With BF16 factors a value
next to a rounding boundary may also fall on the other side of it (a
difference of 2^-8 in one entry of one block): 1e-4, as in the other BF16
apply tests."""
import numpy as np
import pytest

import oracle
import reservoir_inputs as ri

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1701_05913_amd as K  # noqa: E402
from tests.gpu_helpers import GpuSystem, pc_apply, relerr  # noqa: E402

PRECS = [(K.KRY_PREC_F64, "f64", 1e-12), (K.KRY_PREC_F32, "f32", 1e-5),
         (K.KRY_PREC_BF16_FACTORS, "bf16", 1e-4)]
#        TJ = 2 .. 8 with their TK, one tile to many
GRIDS = [(5, 2, 33), (4, 3, 22), (6, 4, 17), (7, 5, 13), (3, 6, 11), (9, 7, 10), (3, 8, 2),
         # step counts around the rings' 4, 16 and 32 slots
         (3, 3, 2), (3, 8, 8), (4, 8, 8), (17, 8, 8), (18, 9, 9), (19, 16, 8), (51, 17, 25),
         # lines longer than a chunk in both directions, ragged in j and k
         (67, 23, 19)]


@pytest.mark.parametrize("prec,name,tol", PRECS)
@pytest.mark.parametrize("kind", ["scalar", "block"])
@pytest.mark.parametrize("grid", GRIDS)
def test_sweep_tilings(grid, kind, prec, name, tol):
    s = ri.scalar_system(*grid, seed=5) if kind == "scalar" else ri.blackoil_system(*grid, seed=5)
    A = oracle.Matrix.from_system(s)
    v = np.random.default_rng(9).standard_normal(A.n)
    ref = oracle.PC(A, "bilu0", name).apply(v)
    g = GpuSystem(s)
    try:
        z1, z2 = pc_apply(g, K.KRY_PC_ILU0, v, prec=prec, layout=K.KRY_SWEEP_GRID, repeat=2)
    finally:
        g.close()
    assert relerr(z1, ref) <= tol
    assert np.array_equal(z1, z2)
