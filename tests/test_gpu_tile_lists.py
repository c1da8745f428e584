"""GPU: the rasterizer of per-tile lists (small_px < 0) on each tile shape, its
stored and recomputed barycentrics, gradients and one-pass image, against the
CPU oracle."""
import functools

import numpy as np
import pytest

import oracle  # noqa: F401
from paper_2405_02508_amd import scenes
from tests.gpu_util import compare, run_gpu, run_oracle, say, to_dev

pytestmark = pytest.mark.gpu

TILES = [(8, 8), (16, 16), (32, 8), (16, 8)]


@functools.lru_cache(maxsize=None)
def case(k):
    s = scenes.make_config(k, small=True)
    g = scenes.image_grad(s, 0)
    return s, g, run_oracle(s, g)


@pytest.mark.parametrize("k", [1, 2, 4, 5])
@pytest.mark.parametrize("tile", TILES)
def test_tile_shapes(k, tile):
    s, g, ref = case(k)
    say(f"[tile lists] config {k} {s.name} tile {tile}")
    got = run_gpu(s, g, tile=tile, small_px=-1)
    assert got["status"][0]["overflow_tiles"] == 0
    compare(got, ref)
    compare(run_gpu(s, g, tile=tile, small_px=-1, store_bary=False), ref, bary=False, grads=False)
    compare(run_gpu(s, g, tile=tile, small_px=-1, bin_cap=64), ref, grads=False)


@pytest.mark.parametrize("mask", [False, True])
@pytest.mark.parametrize("store_bary", [False, True])
@pytest.mark.parametrize("tile", TILES)
def test_one_pass_image(tile, store_bary, mask):
    import torch
    from paper_2405_02508_amd import mer
    s, _, ref = case(4)
    say(f"[tile lists] image, tile {tile} bary {store_bary} mask {mask}")
    ctx = mer.Context(s.views, device="cuda", tile=tile, small_px=-1)
    v, tri, attr = to_dev(s.v), to_dev(s.tri), to_dev(s.attr)
    n, C = ctx.n_px, attr.shape[1] + int(s.append_z)
    tid, depth = torch.empty(n, dtype=torch.int32, device="cuda"), torch.empty(n, device="cuda")
    bary = torch.empty(n, 2, device="cuda") if store_bary else None
    img, two = torch.full((n, C + int(mask)), -7.0, device="cuda"), torch.full((n, C), -7.0, device="cuda")
    ctx.rasterize_interpolate(v, tri, tid, attr, img, depth=depth, bary=bary, append_z=s.append_z, mask=mask)
    assert np.array_equal(tid.cpu().numpy(), ref["tri_id"])
    ctx.interpolate(attr, v, tri, tid, two, bary=bary, append_z=s.append_z)
    assert torch.equal(img[:, :C], two)
    if mask:
        assert torch.equal(img[:, C], (tid >= 0).float())
