"""Timer names of the sweeps inside a CPR application, on a grid stencil and on
a general pattern: each backward sweep counts under the name of its epilogue
(plain, added to a vector, pressure injected), and every name of a 3x3 sweep
has its bytes in the benchmark's table."""
import numpy as np
import pytest

import bench
import reservoir_inputs as ri

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1701_05913_amd as K  # noqa: E402
from tests.gpu_helpers import GpuSystem, pc_apply  # noqa: E402

PRECS = [(K.KRY_PREC_F64, "f64"), (K.KRY_PREC_F32, "f32"), (K.KRY_PREC_BF16_FACTORS, "bf16")]
SWEEPS = 3
# (variant, plain, added, injected) backward sweeps of the full system
VARIANTS = [("PF", 0, 0, 1), ("FP", 1, 0, 0), ("FPF", 1, 1, 0), ("FFPF", 1, 2, 0)]


@pytest.mark.parametrize("layout", ["GRID", "LEVELS"])
@pytest.mark.parametrize("prec,name", PRECS)
@pytest.mark.parametrize("variant,plain,added,injected", VARIANTS)
def test_names(variant, plain, added, injected, prec, name, layout):
    s = ri.blackoil_system(9, 8, 7, seed=1)
    g = GpuSystem(s)
    K.KernelTimingReset()
    K.KernelTimingSelect(None)
    K.KernelTimingSample(1)
    K.KernelTimingEnable(True)
    try:
        pc_apply(g, K.KRY_PC_CPR, np.ones(g.n), prec=prec, cpr=(getattr(K, f"KRY_CPR_{variant}"), SWEEPS),
                 layout=getattr(K, f"KRY_SWEEP_{layout}"))
        K.KernelTimingEnable(False)
        stored = {"bsr3": name, "csr": "f64" if name == "f64" else "f32"}   # pressure factors: never BF16
        count = {kind + end: K.KernelTimingQuery(f"ilu_bwd_{kind}_{stored[kind]}{end}")[0]
                 for kind in stored for end in ("", "_add", "_inject")}
        forward = {kind: K.KernelTimingQuery(f"ilu_fwd_{kind}_{stored[kind]}")[0] for kind in stored}
    finally:
        K.KernelTimingEnable(False)
        K.KernelTimingReset()
        g.close()
    assert count == {"bsr3": plain, "bsr3_add": added, "bsr3_inject": injected,
                     "csr": 1, "csr_add": SWEEPS - 1, "csr_inject": 0}
    assert forward == {"bsr3": plain + added + injected, "csr": SWEEPS}
    assert {f"ilu_bwd_bsr3_{name}{end}" for end in ("", "_add", "_inject")} <= set(bench.algorithmic_bytes(7, 25))
