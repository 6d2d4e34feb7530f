"""The feature adjoint where a listed splat's vector is not finite and no pixel
uses the splat (it lies between pixel centres): the other splats' gradients are
those of a finite vector, bit for bit, at the widths that take pairs two at a
time (4, 20, 24) and one at a time (32), with lists of odd and even length."""
import math

import pytest

import gen
from helpers import to_device

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("tile_cull", [True, False])
@pytest.mark.parametrize("n", [20, 21])
@pytest.mark.parametrize("N", [4, 20, 24, 32])
def test_unused_pairs_leave_the_gradient_alone(N, n, tile_cull):
    from paper_2311_18561_amd.render import (bin_sort, camera_struct, frame_struct, preprocess, render_features,
                                             render_features_bwd)
    W, H = 16, 16
    scene = gen.make_scene(n, 4, sh_degree=0)
    scene["scale"][:] *= 8.0  # each splat covers most of the tile
    scene["mu"][:2] *= 0.1
    scene["opacity"][:] = 0.2 * scene["opacity"] + 0.05
    scene["tau"][:] = 0.5  # at its life peak: the decayed opacity is the opacity
    params = to_device(scene)
    cam, fr = camera_struct(gen.make_camera(W, H)), frame_struct(0.5)
    geom = preprocess(params, n, 0, cam, fr)
    mid = int(geom.depth.argsort()[n // 2])
    geom.xy[mid] = torch.tensor([7.5, 8.5], device="cuda")
    geom.radius[mid] = 1
    geom.tiles[mid] = 1
    geom.conic_op[mid] = torch.tensor([100.0, 0.0, 100.0, 0.5], device="cuda")
    bins = bin_sort(geom, cam, tile_cull=tile_cull)
    assert bins.num_listed() == n
    feats = torch.linspace(-1.0, 1.0, N * n, device="cuda").reshape(n, N)
    _, T, nc = render_features(geom, bins, cam, feats)
    assert (nc > n // 2 + 1).any()  # pixels that use splats behind the changed one
    dout = torch.linspace(0.5, 1.5, N * H * W, device="cuda").reshape(N, H, W)
    results = []
    for value in (1.0, math.nan, math.inf, -math.inf):
        f = feats.clone()
        f[mid, N // 2] = value
        fg = torch.zeros_like(f)
        grads = render_features_bwd(params, n, 0, [(cam, fr, geom, bins, T, nc)], f, [dout], fg)
        results.append([fg, *grads])
    assert all(torch.isfinite(x).all() for x in results[0]) and any(x.any() for x in results[0])
    for r in results[1:]:
        for a, b in zip(results[0], r):
            assert torch.equal(a, b)
