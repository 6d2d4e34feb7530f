"""The SSIM kernels at the edges of their 32 x 32 tiles against the FP64
oracle: one pixel, one short of a tile, a tile, one over, two channels' worth
of ragged tiles, and an image one window wide.  The image's border pixels
stand next to the zero padding in every one of them.

Bars: those of the SSIM tests (24 FP32 roundings of the window sums; those of
(x - y)^2 are no larger than those of x^2 and y^2; the gradient 1e-3 of the
sum of its terms' magnitudes)."""
import numpy as np
import pytest

from helpers import grad_tolerance_report
from test_gpu_ssim import _map_bound

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("C,H,W", [(1, 1, 1), (3, 31, 31), (3, 32, 32), (3, 33, 33), (2, 65, 97), (1, 11, 70),
                                   (1, 70, 11)])
def test_ssim_tile_edges(orc, C, H, W):
    import paper_2311_18561_amd as pvg
    rng = np.random.default_rng(100 * H + W)
    x, y = (rng.random((C, H, W)).astype(np.float32) for _ in range(2))
    g = rng.standard_normal((C, H, W)).astype(np.float32)
    tx = torch.from_numpy(x).cuda().requires_grad_(True)
    S = pvg.pvg_ssim(tx, torch.from_numpy(y).cuda())
    (S * torch.from_numpy(g).cuda()).sum().backward()
    S_ref = orc.ssim.ssim_map(x, y)
    err = np.abs(S.detach().cpu().numpy() - S_ref) / _map_bound(x.astype(np.float64), y.astype(np.float64), S_ref)
    print(f"[{C}x{H}x{W}] map: worst/bound = {err.max():.3g}")
    assert err.max() <= 1.0
    dx, mag = orc.ssim.ssim_grad(x, y, g, magnitude=True)
    worst, l2 = grad_tolerance_report(tx.grad.cpu().numpy(), dx, rel=1e-3, magnitude=mag)
    print(f"[{C}x{H}x{W}] gradient: worst/tol = {worst:.3g}, l2 rel = {l2:.3g}")
    assert worst <= 1.0
