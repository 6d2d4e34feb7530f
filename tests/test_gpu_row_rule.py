"""The lists on either side of the sizes where sorting row records gives way to
sorting instances: a scene of the largest number of Gaussians that takes the
first, and the same scene with one more behind the camera, which takes the
second, have the same keys, values, ranges, row records and first indices."""
import pytest

import gen
from helpers import to_device

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# one pass of the tile id, two passes and up to 512 tiles, more than 256 tile rows of fewer than 8 columns
@pytest.mark.parametrize("W,H,n", [(256, 256, 1 << 17), (320, 240, 3 << 19), (48, 4112, 1 << 19)])
def test_same_lists(W, H, n):
    from paper_2311_18561_amd.render import bin_sort, bin_sort_nosync, camera_struct, frame_struct, preprocess
    scene = gen.make_scene(n + 1, 3, sh_degree=0, layout="path")
    scene["mu"][2, n] = -500.0
    scene["vel"][:, n] = 0.0
    cam, fr = camera_struct(gen.make_camera(W, H, fx=300.0)), frame_struct(0.5)
    got = []
    for m in (n, n + 1):
        params = [p[..., :m].contiguous() for p in to_device(scene)]
        geom = preprocess(params, m, 0, cam, fr)
        for bins in (bin_sort(geom, cam), bin_sort_nosync(geom, cam, 3 * n)):
            count = bins.num_listed()
            rows = torch.clamp(((geom.xy[:, 1] + geom.radius + 15) / 16).floor(), 0, (H + 15) // 16)
            rows = rows - torch.clamp(((geom.xy[:, 1] - geom.radius) / 16).floor(), 0, (H + 15) // 16)
            vis = geom.radius > 0
            num_rows = int(rows[vis].sum().item())
            got.append((count, bins.keys[:count], bins.vals[:count], bins.ranges, bins.rows[:2 * num_rows],
                        bins.first[:n][vis[:n]], bins.row_base[:n][vis[:n]]))
    assert got[0][0] > 10000
    for other in got[1:]:
        assert other[0] == got[0][0]
        for a, b in zip(got[0][1:], other[1:]):
            assert torch.equal(a, b)
