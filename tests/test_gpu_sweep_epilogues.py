"""Grid sweeps inside CPR at the edges of their tiling: right-hand sides in FP32
(cells of 12 and of 4 bytes in the ring), the backward sweep's two epilogues
(added to a vector, pressure injected) in every precision, on tiles narrower
than 8 lines (every TJ from 2 to 7), ragged last tiles and step counts around
the rings' lengths.  PF injects, FPF and FFPF add; the pressure stage is scalar
and adds its later sweeps.

Tolerances: as for single sweeps, times the few sweeps and products of a CPR
application: 1e-10 in FP64 (single sweeps 1e-12), 3e-5 in FP32 (1e-5) and 5e-4
with BF16 factors (1e-4)."""
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

PRECS = [(K.KRY_PREC_F64, "f64", 1e-10), (K.KRY_PREC_F32, "f32", 3e-5),
         (K.KRY_PREC_BF16_FACTORS, "bf16", 5e-4)]
#        TJ = 2 .. 7 with their TK, ragged tiles, rings' lengths
GRIDS = [(5, 2, 33), (4, 3, 22), (6, 4, 17), (7, 5, 13), (3, 6, 11), (9, 7, 10), (3, 3, 2),
         (17, 8, 8), (18, 9, 9), (51, 17, 25)]


@pytest.mark.parametrize("prec,name,tol", PRECS)
@pytest.mark.parametrize("variant", ["PF", "FPF", "FFPF"])
@pytest.mark.parametrize("grid", GRIDS)
def test_cpr_tilings(grid, variant, prec, name, tol):
    s = ri.blackoil_system(*grid, seed=5)
    A = oracle.Matrix.from_system(s)
    v = np.random.default_rng(9).standard_normal(A.n)
    ref = oracle.PC(A, f"cpr_{variant.lower()}", name, p_sweeps=3).apply(v)
    g = GpuSystem(s)
    try:
        z1, z2 = pc_apply(g, K.KRY_PC_CPR, v, prec=prec, cpr=(getattr(K, f"KRY_CPR_{variant}"), 3),
                          layout=K.KRY_SWEEP_GRID, repeat=2)
    finally:
        g.close()
    assert relerr(z1, ref) <= tol
    assert np.array_equal(z1, z2)
