"""GPU: coarse tiles on both sides of the number up to which each has a cache
line of counters, with triangles of every list kind (ranked, tested by 16
lanes, walked, and a list in parts), against the CPU oracle bit for bit."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import say, to_dev
from tests.test_gpu_long_lists import cluster

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,n_tiles", [(2048, 2048, 4096), (2048, 2049, 4160)])
def test_many_tiles(H, W, n_tiles):
    import torch
    from paper_2405_02508_amd import mer
    kinds = [cluster(3000, H, W, (0, 0, W, H), 12.0), cluster(400, H, W, (0, 0, W, H), 150.0),
             cluster(60, H, W, (0, 0, W, H), 1500.0), cluster(9000, H, W, (1000, 1000, 1020, 1020), 10.0)]
    v_np = np.concatenate([k[0] for k in kinds])
    n_t = v_np.shape[0] // 3
    tri_np = np.arange(3 * n_t, dtype=np.int32).reshape(n_t, 3)
    views = np.array([[0, 0, 0, 0, 3 * n_t, n_t, H, W]], np.int64)
    say(f"[many tiles] {n_t} triangles, {W}x{H}")
    ctx = mer.Context(views, device="cuda")
    assert ctx.plan.ct_log2 == 5 and ctx.plan.total_ctiles == n_tiles
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
