"""GPU: the forward-mode tangent of rows that no vector store takes, whose
tiles are 8 x 8 pixels, at the edges of those tiles and at the widths on both
sides of the rule, against the CPU oracle.  Tolerance and the absence of
intersections as in the test of the 16 x 16 tiles' edges."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2405_02508_amd import mer, scenes
from tests.gpu_util import say
from tests.test_gpu_jvp import check, gpu_jvp, tangents

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C", [2, 5, 7, 8, 11, 13, 17])
@pytest.mark.parametrize("W,H", [(1, 1), (7, 9), (8, 8), (9, 8), (25, 17), (47, 49)])
def test_jvp_of_unaligned_rows(W, H, C):
    s = scenes.scattered_triangles(W * 64 + H, 8 + W * H // 24, H, W, 9.0)
    rng = np.random.default_rng(C)
    s = dataclasses.replace(s, attr=rng.uniform(0, 1, size=(s.attr.shape[0], C)).astype(np.float32))
    views = np.repeat(s.views, 2, 0)
    views[1, 3], views[1, 6], views[1, 7] = W * H, W, H  # the same triangles over H x W
    for name, v in (("one view", s.views), ("two views", views)):
        sc = dataclasses.replace(s, views=v)
        say(f"[jvp rows] {W}x{H}, {C} channels, {name}")
        dv, da = tangents(sc, W + H)
        got = gpu_jvp(sc, dv, da, flags=mer.NO_INTERSECT)
        f = oracle.forward(sc)
        assert np.array_equal(got["tid"].cpu().numpy(), f["tri_id"])
        check(got["dimg"].cpu().numpy(), oracle.jvp(sc, f, dv, da, flags=mer.NO_INTERSECT), f"{W}x{H} C {C} {name}")
