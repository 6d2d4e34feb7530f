"""The compositing adjoint's groups of four pairs against the oracle's FP64
adjoint: lists shorter than a group and of every remainder, one tile, ragged
images whose last tiles lie partly outside, both list forms, with and without
the channels' gradients, and with splats that reach the 0.99 clamp (the walk
with the clamp's tests).

Bar: that of the parity tests, 1e-3 of max(|g*|, 1e-2 rms, 1e-2 terms) per
element; pixels with an ambiguous decision carry no loss."""
import numpy as np
import pytest

import gen
from helpers import FIELDS, grad_tolerance_report, oracle_grads, oracle_margin, to_device

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# (width, height, Gaussians): 1, 6 and 12 tiles, then 1,024 and 1,056 tiles of a few pairs each
SIZES = [(7, 5, 200), (33, 17, 800), (61, 47, 2000), (512, 512, 2500), (528, 512, 2500)]


@pytest.mark.parametrize("channels,tile_cull,opaque", [(False, True, False), (False, False, True), (True, True, True)])
@pytest.mark.parametrize("W,H,n", SIZES)
def test_backward_groups(orc, W, H, n, channels, tile_cull, opaque):
    import paper_2311_18561_amd as pvg
    scene = gen.make_scene(n, W + H, sh_degree=1)
    if opaque:  # a tenth of the splats reach the clamp
        pick = np.random.default_rng(5).uniform(size=n) < 0.1
        scene["opacity"][pick] = 1.0
        scene["tau"][pick] = 0.45  # at its life peak at t = 0.45: the decayed opacity is 1
    cam, t, dt = gen.make_camera(W, H), 0.45, 0.05
    pre = orc.preprocess_f32(scene, cam, t, dt)
    bins = orc.bin_sort(pre, cam)
    keep = (oracle_margin(pre, bins, cam, t, dt, gradients=True) >= 1.0).astype(np.float32)
    rng = np.random.default_rng(W)
    w = (rng.standard_normal((3, H, W)) * keep).astype(np.float32)
    wD = (0.05 * rng.standard_normal((H, W)) * keep).astype(np.float32)
    wO = (rng.standard_normal((H, W)) * keep).astype(np.float32)
    wF = (rng.standard_normal((4, H, W)) * keep).astype(np.float32)
    cu = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    params = [p.requires_grad_(True) for p in to_device(scene)]
    kw = {}
    if channels:
        img, depth, opac, vbar, rho = pvg.pvg_render_views(params, [(cam, t, dt)], tile_cull=tile_cull, channels=True)
        loss = ((img[0] * cu(w)).sum() + (depth[0] * cu(wD)).sum() + (opac[0] * cu(wO)).sum()
                + (vbar[0] * cu(wF[:3])).sum() + (rho[0] * cu(wF[3])).sum())
        kw = dict(dD=wD.astype(np.float64), dT=-wO.astype(np.float64), dF=wF.astype(np.float64))
    else:
        img = pvg.pvg_render(params, cam, t, dt, tile_cull=tile_cull)
        loss = (img * cu(w)).sum()
    loss.backward()
    ref, _, terms = oracle_grads(orc, orc.scene64(scene), cam, t, dt, 0, (0.0, 0.0, 0.0), pre, bins,
                                 w.astype(np.float64), **kw)
    for f, p in zip(FIELDS, params):
        worst, l2 = grad_tolerance_report(p.grad.detach().cpu().numpy(), ref[f], rel=1e-3, terms=terms[f])
        print(f"[{W}x{H} channels={channels} cull={tile_cull}] {f}: worst/tol = {worst:.3g}, l2 rel = {l2:.3g}")
        assert worst <= 1.0, f
