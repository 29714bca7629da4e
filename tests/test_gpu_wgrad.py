"""Weight and bias gradients of every layer at the edges of the weight-gradient
kernel's bricks (16 x 4 x 2 cells, the output gradient read one cell further
in x on both sides) and of the reductions' block counts, against the oracle's
BF16 emulation.

Tolerance: operands are the same BF16 values on both sides and the sums FP32
against FP64, so what differs is the rounding of an activation or a gradient
that falls next to a BF16 boundary (2^-9 of that value, here and there): 1e-2
per layer, as for the whole gradient elsewhere; a misplaced cell, channel or
tap changes a layer's gradient by its own size."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1701_05913_amd as K  # noqa: E402
from tests.gpu_helpers import DEV, relerr  # noqa: E402


@pytest.mark.parametrize("grid", [(1, 1, 1), (15, 3, 1), (16, 4, 2), (33, 5, 3), (31, 9, 7), (48, 2, 65)])
def test_layer_gradients_at_brick_edges(grid):
    nx, ny, nz = grid
    cells = nx * ny * nz
    rng = np.random.default_rng(21)
    ch = oracle.CONV_CH
    prm = np.concatenate([np.concatenate([(2.0 * rng.random(co * ci * 27) - 1.0) * 2.0 / np.sqrt(27.0 * ci),
                                          0.1 * rng.standard_normal(co)])
                          for ci, co in zip(ch[:-1], ch[1:])]).astype(np.float32)
    inp = rng.standard_normal(4 * cells).astype(np.float32)
    tgt = rng.standard_normal(3 * cells).astype(np.float32)
    loss_ref, ref = oracle.conv_loss_grad(grid, prm.astype(np.float64), inp.astype(np.float64),
                                          tgt.astype(np.float64), bf16=True)
    L = K.LearnedCreate(nx, ny, nz, True)
    try:
        K.LearnedSetParams(L, prm)
        grad = torch.zeros(K.LearnedNumParams(), dtype=torch.float32, device=DEV)
        loss = K.LearnedLossGrad(L, torch.from_numpy(inp).to(DEV), torch.from_numpy(tgt).to(DEV), grad)
        got = grad.cpu().numpy().astype(np.float64)
    finally:
        K.LearnedDestroy(L)
    assert abs(loss - loss_ref) <= 1e-3 * abs(loss_ref)
    at = 0
    for ci, co in zip(ch[:-1], ch[1:]):
        w, b = co * ci * 27, co
        assert relerr(got[at:at + w], ref[at:at + w]) <= 1e-2
        assert relerr(got[at + w:at + w + b], ref[at + w:at + w + b]) <= 1e-2
        at += w + b
