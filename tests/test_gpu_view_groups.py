"""The per-Gaussian adjoint over several groups of views in one pass.

A pass sums its views three at a time and adds the groups' chains in turn, so
one call over all views must equal, bit for bit, a call per three views that
accumulates: 4, 6, 7 and 8 views (a last group of 1, 3, 1 and 2), 9 and 11
(two passes, as eight views share the scratch), and a change of the render
time inside a group.  Gaussians outside every view get zeros over whatever the
gradient arrays held."""
import pytest

import gen
from helpers import to_device

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _views(params, n, degree, count, split):
    from paper_2311_18561_amd.render import bin_sort, camera_struct, frame_struct, preprocess, render_fwd
    out = []
    for k in range(count):
        cam = camera_struct(gen.yaw_camera(150, 90, -30.0 + 11.0 * k, (0.0, 0.0, 0.0)))
        frame = frame_struct(0.4 if k < split else 0.6, 0.03 * (k % 2))
        geom = preprocess(params, n, degree, cam, frame)
        bins = bin_sort(geom, cam)
        _, final_T, n_contrib = render_fwd(geom, bins, cam, frame)[:3]
        g = torch.Generator(device="cuda").manual_seed(k)
        out.append((cam, frame, geom, bins, final_T, n_contrib, torch.randn((3, 90, 150), device="cuda", generator=g)))
    return out


@pytest.mark.parametrize("count,split", [(4, 99), (6, 99), (7, 99), (8, 99), (9, 99), (11, 99), (6, 2), (8, 4)])
def test_one_pass_equals_a_pass_per_group(count, split):
    from paper_2311_18561_amd.render import render_bwd_views
    n, degree = 4001, 2
    params = to_device(gen.make_scene(n, count, sh_degree=degree))
    views = _views(params, n, degree, count, split)
    whole = [torch.full_like(p, float("nan")) for p in params]
    stats = torch.zeros((2, n), device="cuda")
    render_bwd_views(params, n, degree, views, whole, stats=stats)
    # the groups: three views, cut where the time changes and after every eighth view
    groups, cur = [], []
    for k, v in enumerate(views):
        if cur and (len(cur) == 3 or k % 8 == 0 or k == split):
            groups.append(cur)
            cur = []
        cur.append(v)
    groups.append(cur)
    parts = [torch.empty_like(p) for p in params]
    part_stats = torch.zeros((2, n), device="cuda")
    for q, vs in enumerate(groups):
        render_bwd_views(params, n, degree, vs, parts, accumulate=q > 0, stats=part_stats)
    for a, b in zip(whole, parts):
        assert torch.equal(a, b)
    assert torch.equal(stats, part_stats)
    unseen = torch.stack([v[2].radius for v in views]).eq(0).all(0)
    assert unseen.any() and not unseen.all()
    for p in whole:
        assert not p[..., unseen].any()
