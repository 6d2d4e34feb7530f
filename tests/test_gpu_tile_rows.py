"""Culled lists built by tile rows, against lists rebuilt on the host from the
row records: every visible Gaussian's rows in (depth, index) order, expanded
and stably sorted by tile.  Sizes: one tile; 256, 257, 1,024 and 1,025 tile
rows (the row digits' widths, and the last taken by instance sorting); 255 and
256 columns (the packed keys' limit); records and instances of a tile row past
one chunk (256) and one run (4,096); and capacities too small for the tables.
All outputs are whole numbers and must be equal."""
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


def _u32(t):
    return t.cpu().numpy().view(np.uint32)


def _check(geom, bins, W, H):
    GX, GY = (W + 15) // 16, (H + 15) // 16
    radius = geom.radius.cpu().numpy()
    y = geom.xy.cpu().numpy()[:, 1]
    r = radius.astype(np.float32)
    y0 = np.clip(np.floor((y - r) / np.float32(16)), 0, GY).astype(np.int64)
    y1 = np.clip(np.floor(((y + r) + np.float32(15)) / np.float32(16)), 0, GY).astype(np.int64)
    vis = np.flatnonzero(radius > 0)
    order = vis[np.argsort(geom.depth.cpu().numpy()[vis].view(np.uint32), kind="stable")]
    nrow = (y1 - y0)[order]
    base = np.concatenate(([0], np.cumsum(nrow)))
    row_base, first = _u32(bins.row_base), _u32(bins.first)
    assert np.array_equal(row_base[order], ((base[:-1] - y0[order]) & 0xffffffff).astype(np.uint32))
    rows = _u32(bins.rows)[:2 * base[-1]].reshape(-1, 2)
    ln = (rows[:, 1] >> 16).astype(np.int64)
    off = np.cumsum(ln) - ln
    assert np.array_equal(rows[:, 0], off.astype(np.uint32))
    assert np.array_equal(first[order], off[base[:-1]].astype(np.uint32))
    g = np.repeat(order, nrow)
    ty = np.arange(base[-1]) - np.repeat(base[:-1], nrow) + np.repeat(y0[order], nrow)
    tile = np.repeat(ty * GX + (rows[:, 1] & 0xffff).astype(np.int64) - off, ln) + np.arange(ln.sum())
    s = np.argsort(tile, kind="stable")
    m = int(ln.sum())
    assert bins.num_listed() == m
    assert np.array_equal(_u32(bins.keys)[:m], tile[s].astype(np.uint32))
    assert np.array_equal(_u32(bins.vals)[:m], np.repeat(g, ln)[s].astype(np.uint32))
    cnt = np.bincount(tile, minlength=GX * GY)
    end = np.cumsum(cnt)
    want = np.where(cnt[:, None] > 0, np.stack((end - cnt, end), 1), 0)
    assert np.array_equal(_u32(bins.ranges).reshape(-1, 2), want.astype(np.uint32))
    return m


@pytest.mark.parametrize("W,H,n,grow", [
    (7, 5, 1, 1.0), (16, 16, 700, 1.0), (16, 4096, 900, 1.0), (16, 4112, 900, 1.0), (16, 16384, 900, 1.0),
    (16, 16400, 900, 1.0), (4080, 40, 700, 1.0), (4096, 40, 700, 1.0), (2048, 33, 600, 30.0), (203, 119, 5000, 4.0)])
def test_lists(W, H, n, grow):
    from paper_2311_18561_amd import bin_sort, bin_sort_nosync
    from paper_2311_18561_amd.render import camera_struct, frame_struct, preprocess
    scene = gen.make_scene(n, W + H)
    scene["scale"] *= np.float32(grow)
    cam = camera_struct(gen.make_camera(W, H))
    geom = preprocess(to_device(scene), n, 0, cam, frame_struct(0.5))
    bins = bin_sort(geom, cam)
    m = _check(geom, bins, W, H)
    rows = int(((torch.clamp((geom.xy[:, 1] + geom.radius + 15).div(16).floor(), 0, (H + 15) // 16)
                 - torch.clamp((geom.xy[:, 1] - geom.radius).div(16).floor(), 0, (H + 15) // 16))
                [geom.radius > 0]).sum())
    need = max(m, rows, 1)
    for capacity in (need, need + 1, 4 * need + 5000):  # too small for the tables; enough
        assert _check(geom, bin_sort_nosync(geom, cam, capacity), W, H) == m
    if m > 1:
        over = bin_sort_nosync(geom, cam, max(1, m - 1))  # over capacity: every list empty
        torch.cuda.synchronize()
        assert not over.ranges.any()


@pytest.mark.parametrize("n", [1, 63, 65, 1024, 1025, 3000, 8191, 8192, 8193])
def test_few_gaussians(n):
    """The one-block ordering up to 8,192 Gaussians, and one more: every third
    Gaussian at the depth of another (ties go by index), both list forms, over
    capacity, and nothing in view."""
    from paper_2311_18561_amd import bin_sort, bin_sort_nosync
    from paper_2311_18561_amd.render import camera_struct, frame_struct, preprocess
    scene = gen.make_scene(n, n)
    scene["mu"][:, ::3] = scene["mu"][:, :1]
    for f in ("vel", "period", "tau"):
        scene[f][..., ::3] = scene[f][..., :1]
    W, H = 203, 119
    for seen in (True, False):
        cam = camera_struct(gen.make_camera(W, H))
        if not seen:
            cam.znear = 1e6
        geom = preprocess(to_device(scene), n, 0, cam, frame_struct(0.5))
        vis = np.flatnonzero(geom.radius.cpu().numpy() > 0)
        assert seen or vis.size == 0
        m = _check(geom, bin_sort(geom, cam), W, H)
        assert _check(geom, bin_sort_nosync(geom, cam, 1 << 18), W, H) == m
        if m > 1:
            over = bin_sort_nosync(geom, cam, 1)
            torch.cuda.synchronize()
            assert not over.ranges.any() and int(over.counters[2]) == 1
        rect = bin_sort(geom, cam, tile_cull=False)
        torch.cuda.synchronize()
        count = _u32(geom.tiles).astype(np.int64)
        order = vis[np.argsort(geom.depth.cpu().numpy()[vis].view(np.uint32), kind="stable")]
        first = np.cumsum(count[order]) - count[order]
        assert int(rect.counters[1]) == vis.size and rect.num_listed() == count.sum()
        assert np.array_equal(_u32(rect.first)[order], first.astype(np.uint32))


@pytest.mark.parametrize("spread", [0.0, 1e-6, 1.0, 1e9])
def test_few_gaussians_of_any_depth_range(spread):
    """The one-block sort's digits cover the bits that differ: none, the
    lowest few, the usual three digits, and four."""
    from paper_2311_18561_amd import bin_sort
    from paper_2311_18561_amd.render import camera_struct, frame_struct, preprocess
    n, W, H = 700, 203, 119
    scene = gen.make_scene(n, 3)
    scene["vel"][:] = 0.0
    grow = np.exp(np.random.default_rng(4).uniform(0.0, np.log1p(spread), size=n))
    scene["mu"] = np.float32([[0.1], [0.2], [4.0]]) * grow.astype(np.float32)
    scene["scale"] *= grow.astype(np.float32)
    geom = preprocess(to_device(scene), n, 0, camera_struct(gen.make_camera(W, H)), frame_struct(0.5))
    depth = geom.depth.cpu().numpy()[geom.radius.cpu().numpy() > 0].view(np.uint32)
    differ = int(np.bitwise_or.reduce(depth) & ~np.bitwise_and.reduce(depth))
    width = differ.bit_length() - ((differ & -differ).bit_length() - 1) if differ else 0
    assert {0.0: width == 0, 1e-6: 0 < width <= 9, 1.0: 18 < width <= 27, 1e9: width > 27}[spread]
    _check(geom, bin_sort(geom, camera_struct(gen.make_camera(W, H))), W, H)


def test_batch_of_many_rows():
    """A served batch of 365 tile rows of three widths equals the views rendered alone."""
    import paper_2311_18561_amd as pvg
    from paper_2311_18561_amd.serve import Server
    params = to_device(gen.make_scene(3000, 11, sh_degree=1))
    cams = [gen.make_camera(48, 2400), gen.make_camera(640, 480), gen.make_camera(64, 2960)]
    expect = [pvg.render(params, c, 0.5)[0] for c in cams]
    with Server(max_batch=4, max_inflight=1, max_batch_gaussians=20_000, max_batch_pixels=4 * 640 * 480,
                instance_capacity=1 << 20) as srv:
        sid = srv.load_scene(params)
        outs = [torch.empty_like(e) for e in expect]
        for t in [srv.submit(sid, c, 0.5, o) for c, o in zip(cams, outs)]:
            assert srv.wait(t).status == 0
    for o, e in zip(outs, expect):
        assert torch.equal(o, e)
