"""Dot products around the size up to which one workgroup does them, against
the two-launch form (`VecDotNoAlloc`): the sums run in the same order, so the
results are equal bit for bit; against numpy to 1e-12 of the magnitudes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1701_05913_amd as K  # noqa: E402


@pytest.mark.parametrize("n", [1, 63, 64, 65, 255, 256, 257, 1023, 1025, 2880, 4095, 4096, 4097, 16385])
def test_same_bits(n):
    rng = np.random.default_rng(n)
    x, y = rng.standard_normal(n), rng.standard_normal(n)
    xt, yt = torch.from_numpy(x).to("cuda:0"), torch.from_numpy(y).to("cuda:0")
    out = torch.zeros(1, dtype=torch.float64, device="cuda:0")
    m = K.MapCreateLocal(n)
    xv, yv = K.VecWrap(m, xt), K.VecWrap(m, yt)
    try:
        K.KrylovSetStream(torch.cuda.current_stream())
        d = K.VecDot(xv, yv)
        K.VecDotNoAlloc(xv, yv, out)
        torch.cuda.synchronize()
        assert d == float(out[0].item())
        assert abs(d - float(x @ y)) <= 1e-12 * np.abs(x * y).sum()
        assert K.VecNorm2(xv) == pytest.approx(np.linalg.norm(x), rel=1e-13)
    finally:
        K.VecDestroy(xv)
        K.VecDestroy(yv)
        K.MapDestroy(m)
