"""GPU: a small view's rasterizer without lists, on both sides of the number of
triangles that one workgroup scans, against the CPU oracle bit for bit.  A
view of few tiles and many triangles takes lists: one workgroup scanning them
all took 240 us for 32,000 over 16 x 16 pixels, and the lists take 25."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import say, to_dev
from tests.test_gpu_long_lists import cluster

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_t,H,W,lists", [(2048, 64, 64, False), (2049, 64, 64, True), (20000, 16, 16, True),
                                           (513, 17, 300, False), (2049, 8, 8, True)])
def test_views_of_few_tiles(n_t, H, W, lists):
    import torch
    from paper_2405_02508_amd import mer
    v_np, tri_np, attr_np, views = cluster(n_t, H, W, (0, 0, W, H), 7.0)
    say(f"[direct] {n_t} triangles, {W}x{H}")
    ctx = mer.Context(views, device="cuda")
    v, tri, attr = to_dev(v_np), to_dev(tri_np), to_dev(attr_np)
    n = ctx.n_px
    tid, depth = torch.full((n,), -7, dtype=torch.int32, device="cuda"), torch.full((n,), -7.0, device="cuda")
    out, two, bary = torch.empty(n, 3, device="cuda"), torch.empty(n, 3, device="cuda"), torch.empty(n, 2, device="cuda")
    ctx.rasterize_interpolate(v, tri, tid, attr, out, depth=depth, bary=bary)
    st = ctx.status()
    assert (st["entries"] > 0) == lists and st["overflow_tiles"] == 0
    ref = oracle.rasterize(v_np, tri_np, H, W)
    assert np.array_equal(tid.cpu().numpy(), ref)
    ref_depth = oracle.resolve(v_np, tri_np, H, W, ref)[0]
    assert np.all(np.abs(depth.cpu().numpy() - ref_depth) <= 1e-5 * np.maximum(1, np.abs(ref_depth)))
    ctx.interpolate(attr, v, tri, tid, two, bary=bary)
    assert torch.equal(out, two)
