"""The forward walk on whole, half and quarter tiles (chosen by the image's
tile count) against the FP32 oracle, at the counts where the choice changes,
on ragged images, and with splats that need the 0.99 clamp (opacity 1)
beside ordinary ones, so that batches take both forms of the walk.

Bars: those of the parity tests, the image within 1e-4 of the oracle at every
pixel whose skip and stop decisions are unambiguous and the last contributor
equal there; culled and rectangle lists give the same image bit for bit, and
so do the channel kernels."""
import numpy as np
import pytest

import gen
from helpers import gpu_forward, image_parity, last_contributor_ids, oracle_margin

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# (width, height, Gaussians): 1 x 1 to 4 tiles, 1,024 / 1,056 tiles (quarters to halves), 4,096 / 4,160 (halves to whole)
SIZES = [(7, 5, 300), (33, 17, 1500), (61, 47, 3000), (512, 512, 6000), (528, 512, 6000), (1023, 1017, 8000),
         (1040, 1024, 8000)]


@pytest.mark.parametrize("opaque", [False, True])
@pytest.mark.parametrize("W,H,n", SIZES)
def test_forward_split(orc, W, H, n, opaque):
    import paper_2311_18561_amd as pvg
    scene = gen.make_scene(n, W + H, sh_degree=1)
    if opaque:  # a tenth of the splats reach the clamp
        rng = np.random.default_rng(5)
        pick = rng.uniform(size=n) < 0.1
        scene["opacity"][pick] = 1.0
        scene["tau"][pick] = 0.5  # at its life peak at t = 0.5: the decayed opacity is 1
    cam, fr = gen.make_camera(W, H), (0.5, 0.0, 0, (0.1, 0.2, 0.3))
    o = orc.render(scene, cam, *fr)
    g = gpu_forward(scene, cam, *fr)
    r = gpu_forward(scene, cam, *fr, params=g["_params"], tile_cull=False)
    margin = oracle_margin(o["pre"], o["bins"], cam, *fr)
    amb = margin < 1.0
    err, excused = image_parity(g["img"], o["img"], margin)
    image_parity(g["final_T"], o["final_T"], margin)
    ids = last_contributor_ids(g["n_contrib"], g["vals"], g["ranges"], W)
    ids_orc = last_contributor_ids(o["n_contrib"], o["bins"]["inst_gauss"], o["bins"]["ranges"], W)
    assert not np.any((ids != ids_orc) & ~amb)
    print(f"[{W}x{H}] opaque={opaque} error {err:.3g}, ambiguous {int(amb.sum())}, excused {excused}")
    assert np.array_equal(g["img"], r["img"]) and np.array_equal(g["final_T"], r["final_T"])
    imgs, *_ = pvg.pvg_render_views(g["_params"], [(cam, *fr)], channels=True)
    assert np.array_equal(imgs[0].cpu().numpy(), g["img"])
