"""The feature adjoint's pairs of pairs (widths up to 24) and single pairs (32)
on lists of odd and even length, a ragged image whose last tiles lie partly
outside, and splats that reach the 0.99 clamp (the walk with the clamp's
tests): the comparison and the bars of the semantic tests."""
import pytest

import gen
from test_gpu_semantic import _needs_gpu, test_semantic_vs_fp64 as compare  # noqa: F401

pytestmark = pytest.mark.gpu


def _scene(n, opaque):
    scene = gen.make_scene(n, n, sh_degree=1)
    if opaque:  # at its life peak at t = 0.45: the decayed opacity is 1
        scene["opacity"][::5] = 1.0
        scene["tau"][::5] = 0.45
    return scene


@pytest.mark.parametrize("N", [4, 20, 24, 32])
@pytest.mark.parametrize("n,opaque", [(1, False), (150, True), (301, False)])
def test_pair_groups(orc, n, opaque, N):
    compare(orc, f"n={n} opaque={opaque}", lambda: _scene(n, opaque),
            lambda: gen.yaw_camera(37, 21, 5.0, (0.1, 0.0, -0.3)), 0.45, N)
