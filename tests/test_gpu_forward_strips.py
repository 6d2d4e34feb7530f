"""The forward walk's strips (tiles of small images split over two or four
waves) on long thin splats: a strip may leave out only pairs that none of its
pixels uses.  The feature walk takes whole tiles and decides pair by pair as
the colour walk does, so final_T and n_contrib of the two renders are equal bit
for bit.  Splats are 300 to 4,000 pixels long and about a pixel wide, where
rounding of the conic's quadratic form is of the size of its minimum."""
import numpy as np
import pytest

import gen
from helpers import to_device

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def needles(n, seed, fx):
    """n splats whose screen sizes are log-uniform over 300 to 4,000 pixels by
    a few tenths of one, turned about the view axis, with low opacities."""
    rng = np.random.default_rng(seed)
    scene = gen.make_scene(n, seed, sh_degree=0)
    z = scene["mu"][2].astype(np.float64)
    scene["scale"][0] = np.exp(rng.uniform(np.log(300.0), np.log(4000.0), n)) * z / fx
    scene["scale"][1:] = rng.uniform(0.02, 0.8, (2, n)) * z / fx
    half = rng.uniform(0.0, np.pi, n)
    scene["rot"][:] = np.stack([np.cos(half), np.zeros(n), np.zeros(n), np.sin(half)])
    scene["opacity"][:] = rng.uniform(0.01, 0.1, n)
    scene["tau"][:] = 0.5  # at its life peak: the decayed opacity is the opacity
    return scene


@pytest.mark.parametrize("tile_cull", [True, False])
@pytest.mark.parametrize("W,H", [(512, 512), (201, 139), (640, 480), (960, 640)])
def test_strips_keep_every_used_pair(W, H, tile_cull):
    from paper_2311_18561_amd.render import (bin_sort, camera_struct, frame_struct, preprocess, render_features,
                                             render_fwd)
    n = 12000
    cam = gen.make_camera(W, H)
    params = to_device(needles(n, W, cam["fx"]))
    c, fr = camera_struct(cam), frame_struct(0.5)
    geom = preprocess(params, n, 0, c, fr)
    bins = bin_sort(geom, c, tile_cull=tile_cull)
    _, final_T, n_contrib = render_fwd(geom, bins, c, fr)
    _, feat_T, feat_n = render_features(geom, bins, c, torch.ones((n, 4), device="cuda"))
    assert (n_contrib > 0).float().mean() > 0.5
    print(f"[{W}x{H}] cull={tile_cull}: T differs at {(final_T != feat_T).sum().item()} pixels by up to "
          f"{(final_T - feat_T).abs().max().item():.3g}, n_contrib at {(n_contrib != feat_n).sum().item()}")
    assert torch.equal(final_T, feat_T)
    assert torch.equal(n_contrib, feat_n)
