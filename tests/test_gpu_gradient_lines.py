"""GPU parity of the gradient's passes over lines held in LDS, where they can
go wrong: a line of one sample, lines that end inside a group of four, the
column count of a block's last lines, columns just past the segmented range,
images whose lines take several waves of blocks, and lines too long for LDS
(passes from global memory), against float64 within the tolerance derived in
test_gpu_gradient.py (2e-5 of the largest magnitude)."""
import numpy as np
import pytest

from oracle import deriche
from paper_1603_09180_amd import thin

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL = 2e-5


@pytest.mark.parametrize("h,w,dt", [(1, 1, np.uint8), (1, 6, np.uint16), (6, 1, np.uint8),
                                    (5, 2, np.uint8), (33, 13, np.uint16), (1025, 5, np.uint8),
                                    (1026, 258, np.uint16), (1030, 1025, np.uint8),
                                    (1603, 1283, np.uint8), (2600, 300, np.uint8),
                                    (300, 2600, np.uint16), (11000, 9, np.uint8),
                                    (9, 11000, np.uint8), (3100, 2900, np.uint8)])
def test_lines(h, w, dt):
    rng = np.random.default_rng(h * 100003 + w)
    F = rng.integers(0, int(np.iinfo(dt).max) + 1, size=(h, w)).astype(dt)
    alpha, gain = 0.75, 0.5
    print("case gradient lines", h, w, np.dtype(dt).name, flush=True)
    src = torch.from_numpy(F).cuda()
    dst = torch.empty((h, w), dtype=torch.uint16, device="cuda")
    mag = torch.empty((h, w), dtype=torch.float32, device="cuda")
    with thin.Context() as ctx:
        ctx.gradient(src, dst, alpha, gain, magnitude=mag)
    torch.cuda.synchronize()
    _, _, m64 = deriche.gradient(F, alpha)
    tol = TOL * max(float(m64.max()), float(F.max()), 1.0)
    assert float(np.abs(mag.cpu().numpy().astype(np.float64) - m64).max()) <= tol
    q64, margin = deriche.quantize_reference(m64, gain, np.uint16)
    diff = np.abs(dst.cpu().numpy().astype(np.int64) - q64.astype(np.int64))
    near = margin <= tol * gain + 2.0 ** -23 * (m64 * gain + 1.0)
    assert not diff[~near].any()
    assert int(diff.max()) <= max(1, int(np.ceil(2 * tol * gain)))
