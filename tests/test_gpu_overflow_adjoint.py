"""The adjoints over lists of a sort that overflowed without the host count:
they hold nothing, and the index arrays (first[], rows, row_base), which such a
sort does not write, may hold anything; the gradients are zero."""
import pytest

import gen
from helpers import to_device

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("garbage", [-15, 17, 0x7ffffff1])
@pytest.mark.parametrize("tile_cull", [True, False])
def test_gradients_are_zero(tile_cull, garbage):
    from paper_2311_18561_amd.render import (bin_sort_nosync, camera_struct, frame_struct, preprocess, render_bwd,
                                             render_features_bwd, render_fwd)
    n, W, H, nch = 1000, 80, 48, 4
    params = to_device(gen.make_scene(n, 3, sh_degree=1))
    cam, frame = camera_struct(gen.make_camera(W, H)), frame_struct(0.5)
    geom = preprocess(params, n, 1, cam, frame)
    bins = bin_sort_nosync(geom, cam, 100, tile_cull)
    _, final_T, n_contrib = render_fwd(geom, bins, cam, frame)
    assert bins.counters[2].item() == 1 and not n_contrib.any()
    for x in (bins.first, bins.rows, bins.row_base):
        x.fill_(garbage)
    grads = render_bwd(params, n, 1, cam, frame, geom, bins, final_T, n_contrib, torch.ones((3, H, W), device="cuda"))
    assert not any(g.any().item() for g in grads)
    feats, feat_grad = torch.ones((n, nch), device="cuda"), torch.zeros((n, nch), device="cuda")
    grads = render_features_bwd(params, n, 1, [(cam, frame, geom, bins, final_T, n_contrib)], feats,
                                [torch.ones((nch, H, W), device="cuda")], feat_grad)
    assert not feat_grad.any() and not any(g.any().item() for g in grads)
