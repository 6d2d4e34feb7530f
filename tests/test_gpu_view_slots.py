"""The per-Gaussian adjoint where the render time changes at the view that
takes the last of the eight gradient slots, with views enough behind it to
take that slot again: the gradients of one call equal, bit for bit, those of a
call per group that accumulates.  Eight views before the change are two whole
groups of three and one of two; (16, 8) changes on the first slot again."""
import pytest

import gen
from helpers import to_device
from test_gpu_view_groups import _needs_gpu, _views  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# (views, the view the time changes at, the groups' first views)
CASES = [(16, 7, (0, 3, 6, 7, 10, 13)), (17, 7, (0, 3, 6, 7, 10, 13, 16)), (16, 8, (0, 3, 6, 8, 11, 14))]


@pytest.mark.parametrize("count,split,firsts", CASES)
def test_time_change_at_the_last_slot(count, split, firsts):
    from paper_2311_18561_amd.render import render_bwd_views
    n, degree = 2001, 1
    params = to_device(gen.make_scene(n, count, sh_degree=degree))
    views = _views(params, n, degree, count, split)
    whole = [torch.full_like(p, float("nan")) for p in params]
    stats = torch.zeros((2, n), device="cuda")
    render_bwd_views(params, n, degree, views, whole, stats=stats)
    parts = [torch.empty_like(p) for p in params]
    part_stats = torch.zeros((2, n), device="cuda")
    for a, b in zip(firsts, firsts[1:] + (count,)):
        render_bwd_views(params, n, degree, views[a:b], parts, accumulate=a > 0, stats=part_stats)
    for x, y in zip(whole, parts):
        assert torch.isfinite(x).all() and torch.equal(x, y)
    assert torch.equal(stats, part_stats)
