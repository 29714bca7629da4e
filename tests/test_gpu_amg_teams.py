"""AMG V-cycle where its launches change shape: coarse levels whose last chunk
is not whole, one smoothing sweep (the restriction then does all of the way
down's smoothing), two levels (the restriction smooths nothing), every chunk
size, levels of a few rows and levels wide enough for every team size.

Tolerance: as in the other V-cycle comparisons, the sums differ from the
oracle's by their order alone: 1e-11."""
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


@pytest.mark.parametrize("chunk", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("grid,levels,sweeps", [((7, 5, 3), 8, 2), ((19, 13, 7), 8, 1), ((19, 13, 7), 2, 2),
                                                ((33, 31, 17), 5, 2), ((70, 61, 31), 8, 1)])
def test_vcycle_shapes(grid, levels, sweeps, chunk):
    s = ri.scalar_system(*grid, seed=6, perm="layered")
    A = oracle.Matrix.from_system(s)
    v = np.random.default_rng(8).standard_normal(A.n)
    ref = oracle.PC.amg(A, max_levels=levels, num_sweeps=sweeps, gs_chunk=chunk).apply(v)
    g = GpuSystem(s)
    try:
        z1, z2 = pc_apply(g, K.KRY_PC_AMG, v, solver=K.KRY_GMRES, amg=(levels, sweeps, chunk), repeat=2)
    finally:
        g.close()
    assert relerr(z1, ref) <= 1e-11
    assert np.array_equal(z1, z2)
