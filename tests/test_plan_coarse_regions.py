"""The workspace regions of the coarse tiles, which mer_plan does not name: they
follow the last one it names, and hold what the kernels index, as the regions
that the count pass and the parts of long lists share with the per-tile lists
do.  No GPU needed."""
import os

import numpy as np
import pytest

from paper_2405_02508_amd import mer
from tests.test_abi import _full_views, _regions, _tiles

COUNT_BYTES, TILE_BYTES, ITEM_BYTES, ENTRY_BYTES = 8, 16, 32, 8  # int2, CTile, CItem, uint2
KEY_BYTES = 8


@pytest.fixture(scope="module", autouse=True)
def built():
    if not os.path.exists(mer.LIB_PATH):
        from paper_2405_02508_amd import build
        build.build()


def align256(x):
    return (x + 255) & ~255


def _one(H, W, n_t):
    return np.array([[0, 0, 0, 0, 3, n_t, H, W]], np.int64)


def parts(n_t):
    """(entries per part, parts) that a plan of n_t triangles has room for."""
    item = align256(n_t // 2048) if n_t > 2048 * 1024 else 1024
    return item, (2 * n_t // item + 7) // 8 * 8 if n_t > 4096 else 0


VIEWS = {
    "one_px": lambda: _one(1, 1, 0), "no_triangles": lambda: _one(640, 480, 0), "short": lambda: _one(300, 200, 4096),
    "first_parts": lambda: _one(300, 200, 4097), "fine": lambda: _one(500, 300, 200000),
    "millions": lambda: _one(2048, 2048, 2097152), "more": lambda: _one(2048, 2048, 2097153),
    "padded": lambda: _one(2048, 2048, 786432), "sparse": lambda: _one(2048, 2048, 786431),
    "packed": lambda: _one(2048, 2049, 900000),
    "head": lambda: _full_views(3), "pair": lambda: _full_views(4), "batch": lambda: _full_views(5),
}


@pytest.mark.parametrize("tile", [(8, 8), (32, 8)])
@pytest.mark.parametrize("name", sorted(VIEWS))
def test_coarse_regions_hold_what_the_kernels_index(name, tile):
    V = VIEWS[name]()
    P = mer.plan_init(V, tile)
    side = 1 << P.ct_log2
    assert side in (8, 16, 32) and P.total_ctiles == _tiles(V, side, side)
    regs = sorted(_regions(P), key=lambda r: r[1])
    _, off, size = regs[-1]  # the last region that the plan names
    assert off == P.off_bigflat
    item, n = parts(int(P.total_tris))
    assert n <= 4096 + 8 and (n == 0 or n * item > 2 * P.total_tris - item)
    # few tiles' counters have a line each, where there are many triangles for each
    line = 128 // COUNT_BYTES if P.total_ctiles <= 4096 and P.total_tris >= 192 * P.total_ctiles else 1
    for more in (P.total_ctiles * COUNT_BYTES * line, P.total_ctiles * TILE_BYTES, n * ITEM_BYTES):
        off, size = align256(off + size), more
    assert P.ws_bytes == align256(off + size)
    # shared regions: a workgroup's entries, eight a triangle, in the set-up
    # records; their number per workgroup, in the large lists' lengths; the
    # large triangles, in their flat list; the keys of split tiles, by pixel
    have = {name: size for name, _, size in regs}
    groups = -(-int(P.total_tris) // 256)
    assert P.n_bingroups == groups
    last = int(P.total_tris) - 256 * max(groups - 1, 0)
    assert have["rec"] >= ((groups - 1) * 8 * 256 + 8 * last) * ENTRY_BYTES if groups else True
    assert have["bign"] >= groups * 4 and have["bigflat"] >= P.total_tris * 4
    assert have["key"] >= (P.total_px - P.px_begin) * KEY_BYTES


def test_per_tile_plans_reserve_no_coarse_tiles():
    V = _one(700, 500, 9000)
    P, C = mer.plan_init(V, small_px=-1), mer.plan_init(V)
    assert P.ws_bytes == align256(P.off_bigflat + P.total_tris * 4) < C.ws_bytes
    assert P.total_ctiles == 0 and P.big_tiles == 16
