"""GPU: coarse tiles whose counters have a cache line each and ones whose
counters lie together, with triangles of every list kind (ranked, tested by 16
lanes, walked, and a list in parts), against the CPU oracle bit for bit."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import say, to_dev
from tests.test_gpu_long_lists import cluster

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,small,ctl,n_tiles", [(160, 160, 70000, 3, 400), (160, 157, 40000, 3, 400),
                                                   (2048, 2049, 3000, 5, 4160)])
def test_counters_apart_and_together(H, W, small, ctl, n_tiles):
    import torch
    from paper_2405_02508_amd import mer
    u = 1 << ctl  # a tile
    kinds = [cluster(small, H, W, (0, 0, W, H), 4.0), cluster(400, H, W, (0, 0, W, H), 4.0 * u),
             cluster(60, H, W, (0, 0, W, H), 30.0 * u), cluster(9000, H, W, (W // 2, H // 2, W // 2 + u, H // 2 + u), 10.0)]
    v_np = np.concatenate([k[0] for k in kinds])
    n_t = v_np.shape[0] // 3
    tri_np = np.random.default_rng(1).permutation(3 * n_t // 3).astype(np.int32)[:, None] * 3 + np.arange(3, dtype=np.int32)
    tri_np = np.ascontiguousarray(tri_np, np.int32)
    views = np.array([[0, 0, 0, 0, 3 * n_t, n_t, H, W]], np.int64)
    say(f"[counters] {n_t} triangles, {W}x{H}")
    ctx = mer.Context(views, device="cuda")
    assert ctx.plan.ct_log2 == ctl and ctx.plan.total_ctiles == n_tiles
    v, tri = to_dev(v_np), to_dev(tri_np)
    tid, depth = torch.empty(ctx.n_px, dtype=torch.int32, device="cuda"), torch.empty(ctx.n_px, device="cuda")
    ref = oracle.rasterize(v_np, tri_np, H, W)
    for _ in range(2):
        tid.fill_(-7)
        ctx.rasterize(v, tri, tid, depth)
        st = ctx.status()
        assert st["overflow_tiles"] == 0 and st["entries"] > 9000
        assert int(ctx.ws[ctx.plan.off_status:ctx.plan.off_status + 64].view(torch.int64)[3]) > 1  # a list in parts
        assert np.array_equal(tid.cpu().numpy(), ref)
