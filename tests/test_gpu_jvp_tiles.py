"""GPU: the forward-mode tangent at the edges of its 16 x 16 tiles, against
the CPU oracle: views of one pixel, one row, one column, a whole tile, a
remainder of one on either side, and a pair of views, so that every pair of
pixels across a tile's side and every missing neighbour is met.

Tolerance: the bars of the forward-mode parity test (relative L2 1e-5 per
tangent image, every element within 1e-4 of the image's largest magnitude),
for the same reasons.  Intersections are left out: at random depths their
denominators come arbitrarily near zero, so that binary32 holds no relative
bar."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2405_02508_amd import mer, scenes
from tests.gpu_util import say
from tests.test_gpu_jvp import check, gpu_jvp, tangents

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H", [(1, 1), (37, 1), (1, 37), (16, 16), (17, 15), (32, 33), (47, 49)])
def test_jvp_at_tile_edges(W, H):
    s = scenes.scattered_triangles(W * 64 + H, 8 + W * H // 24, H, W, 9.0)
    views = np.repeat(s.views, 2, 0)
    views[1, 3], views[1, 6], views[1, 7] = W * H, W, H  # the same triangles over H x W
    for name, v in (("one view", s.views), ("two views", views)):
        sc = dataclasses.replace(s, views=v)
        say(f"[jvp] {W}x{H}, {name}")
        dv, da = tangents(sc, W + H)
        got = gpu_jvp(sc, dv, da, flags=mer.NO_INTERSECT)
        f = oracle.forward(sc)
        assert np.array_equal(got["tid"].cpu().numpy(), f["tri_id"])
        check(got["dimg"].cpu().numpy(), oracle.jvp(sc, f, dv, da, flags=mer.NO_INTERSECT), f"{W}x{H} {name}")
