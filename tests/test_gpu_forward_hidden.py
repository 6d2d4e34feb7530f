"""Splats behind the ones where every pixel of the tile has stopped are not
blended, whatever their records hold: four opaque splats end the walk at the
third, and colours, depths and channels of NaN or infinity from the fifth on
leave image, channels, final_T and n_contrib as finite ones do.  One tile (its
strips go to four waves), 1,056 tiles (two) and 4,225 (one)."""
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


@pytest.mark.parametrize("channels", [False, True])
@pytest.mark.parametrize("W,H", [(16, 16), (528, 512), (1040, 1040)])
def test_hidden_records(W, H, channels):
    from paper_2311_18561_amd.render import bin_sort, camera_struct, frame_struct, preprocess, render_fwd
    n = 12
    params = to_device(gen.make_scene(n, 2, sh_degree=0))
    cam, fr = camera_struct(gen.make_camera(W, H)), frame_struct(0.5)
    geom = preprocess(params, n, 0, cam, fr, feat=True)
    geom.xy.copy_(torch.tensor([0.5 * W, 0.5 * H]).expand(n, 2))
    geom.radius.fill_(2 * max(W, H))
    geom.tiles.fill_(((W + 15) // 16) * ((H + 15) // 16))
    geom.depth.copy_(torch.linspace(1.0, 2.0, n))
    flat = 1e-4 / max(W, H) ** 2  # alpha = o to four digits over the whole image
    geom.conic_op.copy_(torch.tensor([flat, 0.0, flat, 0.98]).expand(n, 4))
    geom.rgb.copy_(torch.linspace(0.1, 0.9, 3 * n).reshape(n, 3))
    geom.feat.copy_(torch.linspace(-1.0, 1.0, 4 * n).reshape(n, 4))
    bins = bin_sort(geom, cam)
    assert bins.num_listed() == n * int(geom.tiles[0])

    def render():
        kw = {}
        if channels:
            kw = {"depth": torch.empty((H, W), device="cuda"), "vbar": torch.empty((3, H, W), device="cuda"),
                  "rho": torch.empty((H, W), device="cuda")}
        return [*render_fwd(geom, bins, cam, fr, **kw), *kw.values()]
    ref = render()
    assert (ref[2] == 2).all() and all(torch.isfinite(x).all() for x in ref)
    for first in (4, 5, 7, 8):
        for value in (math.nan, math.inf):
            geom.rgb[first:] = value
            geom.feat[first:] = value
            geom.depth[first:] = value
            for a, b in zip(ref, render()):
                assert torch.equal(a, b), (first, value)
