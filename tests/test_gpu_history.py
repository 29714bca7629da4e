"""The residual history that the host reads while GMRES runs, step by step
against the oracle's, over two restarts and a part of a third: a budget of
steps and no tolerance, so both take the same number.  Restarts at the edges
of the column counts that the kernels are made for, both forms of
Gram-Schmidt, stored directions (FGMRES) and augmented cycles (LGMRES).

Tolerances: iterates of the same Krylov method on a well-conditioned system
(ILU(0) of the scalar operator), whose estimates differ by rounding times a
modest factor: 1e-9 of the first entry; x by that rounding (some 1e-12) times
the operator's condition (some 1e4): 1e-7.  Three quarters of the steps have to
change the estimate by more than the tolerance, so that a stale or a swapped
entry is seen."""
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

CASES = [("AUTO", K.KRY_GMRES, 0), ("CGS2", K.KRY_GMRES, 0), ("AUTO", K.KRY_FGMRES, 0), ("AUTO", K.KRY_GMRES, 2)]


@pytest.mark.parametrize("ortho,kind,aug", CASES)
@pytest.mark.parametrize("grid,restart", [((5, 3, 2), 1), ((13, 11, 7), 2), ((17, 15, 3), 8), ((16, 14, 6), 9),
                                          ((16, 14, 12), 16), ((19, 18, 15), 17), ((24, 20, 18), 31),
                                          ((24, 20, 18), 32)])
def test_every_entry(grid, restart, ortho, kind, aug):
    s = ri.scalar_system(*grid, seed=11, acc=1e-2)
    A = oracle.Matrix.from_system(s)
    steps = 2 * restart + max(1, restart // 3)
    pc = oracle.PC(A, "bilu0")
    if aug:
        steps = 2 * restart + aug
        ref = oracle.lgmres(A, pc, s["b"], rtol=0.0, restart=restart, aug_k=aug, maxit=steps, hist=True)
    else:
        ref = oracle.gmres(A, pc, s["b"], rtol=0.0, restart=restart, maxit=steps,
                           flexible=kind == K.KRY_FGMRES, hist=True)
    g = GpuSystem(s)
    try:
        gpu = solve(g, kind, K.KRY_PC_BILU0, rtol=0.0, maxit=steps, restart=restart, aug_k=aug,
                    ortho=getattr(K, f"KRY_ORTHO_{ortho}"))
    finally:
        g.close()
    h, r = np.asarray(gpu["hist"]), np.asarray(ref["hist"])
    assert gpu["iters"] == ref["iters"] == steps
    assert h.size == r.size == steps + 1
    apart = np.abs(np.diff(r)) > 4e-9 * r[0]
    assert apart.sum() >= 0.75 * steps
    assert np.max(np.abs(h - r)) <= 1e-9 * r[0]
    assert relerr(gpu["x"], ref["x"]) <= 1e-7
