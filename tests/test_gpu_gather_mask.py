"""The per-Gaussian gather's flag mask: Gaussians with 1 to 48 listed pairs,
whose ranges start at every offset from a 16-byte boundary, gathered by one
thread, and longer ones by a wave.  Every splat covers a block of tiles of a
chosen size and is the only one there or lies behind one that hides it in some
of them, so that flags are set, cleared and mixed.  Against the oracle's FP64
adjoint.

Bar: that of the parity tests, 1e-3 of max(|g*|, 1e-2 rms, 1e-2 terms)."""
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


@pytest.mark.parametrize("channels", [False, True])
@pytest.mark.parametrize("seed", [1, 2])
def test_gather_of_short_ranges(orc, channels, seed):
    import paper_2311_18561_amd as pvg
    W, H, n = 208, 176, 400
    scene = gen.make_scene(n, seed, sh_degree=1)
    grow = np.random.default_rng(seed).choice([0.3, 1.0, 3.0, 8.0], size=n).astype(np.float32)
    scene["scale"] *= grow
    cam, t, dt = gen.make_camera(W, H), 0.45, 0.05
    pre = orc.preprocess_f32(scene, cam, t, dt)
    bins = orc.bin_sort(pre, cam)
    keep = (oracle_margin(pre, bins, cam, t, dt, gradients=True) >= 1.0).astype(np.float32)
    rng = np.random.default_rng(seed)
    w = (rng.standard_normal((3, H, W)) * keep).astype(np.float32)
    wO = (rng.standard_normal((H, W)) * keep).astype(np.float32)
    cu = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    params = [p.requires_grad_(True) for p in to_device(scene)]
    kw = {}
    if channels:
        img, _, opac, _, _ = pvg.pvg_render_views(params, [(cam, t, dt)], channels=True)
        loss = (img[0] * cu(w)).sum() + (opac[0] * cu(wO)).sum()
        kw = dict(dT=-wO.astype(np.float64))
    else:
        loss = (pvg.pvg_render(params, cam, t, dt) * cu(w)).sum()
    loss.backward()
    _, _, _, geom, lists = pvg.render([p.detach() for p in params], cam, t, dt)
    ln = lists.rows.cpu().numpy().view(np.uint32).reshape(-1, 2)[:, 1] >> 16
    base = lists.row_base.cpu().numpy().view(np.uint32).astype(np.int64)
    y = geom.xy.cpu().numpy()[:, 1]
    r = geom.radius.cpu().numpy()
    y0, y1 = (np.clip(np.floor((y + s) / 16), 0, H // 16).astype(np.int64) for s in (-r, r + 15))
    counts = np.array([ln[(base[g] + y0[g]) % 2**32:(base[g] + y1[g]) % 2**32].sum() for g in np.flatnonzero(r > 0)])
    starts = np.array([lists.first[g].item() % 16 for g in np.flatnonzero(r > 0)])
    assert (counts == 1).any() and ((counts > 16) & (counts <= 48)).any() and (counts > 48).any()
    assert len(set(starts)) == 16
    ref, _, terms = oracle_grads(orc, orc.scene64(scene), cam, t, dt, 0, (0.0, 0.0, 0.0), pre, bins,
                                 w.astype(np.float64), **kw)
    for f, p in zip(FIELDS, params):
        worst, l2 = grad_tolerance_report(p.grad.detach().cpu().numpy(), ref[f], rel=1e-3, terms=terms[f])
        print(f"[channels={channels} seed={seed}] {f}: worst/tol = {worst:.3g}, l2 rel = {l2:.3g}")
        assert worst <= 1.0, f
