"""One GMRES cycle at the sizes where the Arnoldi step's launches change:
fewer unknowns than a block's rows, one more or less than a tile of 256, grids
at their limit; restarts at the edges of the column counts the kernels are
made for (8, 16, 32, 64), with both forms of Gram-Schmidt; the residual
history the host reads while the steps run.

Tolerances: iterates after a fixed number of steps of the same Krylov method
on a well-conditioned system (ILU(0) of the accumulation-dominated scalar
operator) differ by rounding times a modest factor: 1e-9; the history's
estimates, |g_{j+1}| relative to |b|: 1e-9 of the first."""
import numpy as np
import pytest

import oracle
import reservoir_inputs as ri

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1701_05913_amd as K  # noqa: E402
from tests.gpu_helpers import GpuSystem, relerr, solve  # noqa: E402


@pytest.mark.parametrize("ortho", ["AUTO", "CGS2"])
@pytest.mark.parametrize("grid,restart", [((1, 1, 1), 4), ((5, 3, 1), 8), ((17, 15, 1), 9), ((16, 4, 4), 16),
                                          ((257, 1, 1), 17), ((9, 19, 6), 31), ((9, 19, 6), 32),
                                          ((12, 11, 9), 63), ((64, 48, 45), 12)])
def test_fixed_steps(grid, restart, ortho):
    s = ri.scalar_system(*grid, seed=11, acc=1.0)
    A = oracle.Matrix.from_system(s)
    steps = restart + 2
    ref = oracle.gmres(A, oracle.PC(A, "bilu0"), s["b"], rtol=1e-13, restart=restart, maxit=steps)
    g = GpuSystem(s)
    try:
        gpu = solve(g, K.KRY_GMRES, K.KRY_PC_BILU0, rtol=1e-13, maxit=steps, restart=restart,
                    ortho=getattr(K, f"KRY_ORTHO_{ortho}"))
    finally:
        g.close()
    assert relerr(gpu["x"], ref["x"]) <= 1e-9
    h = np.asarray(gpu["hist"])
    assert h.size == gpu["iters"] + 1
    assert np.all(np.isfinite(h)) and np.all(h[1:] <= h[0] * (1 + 1e-9))
