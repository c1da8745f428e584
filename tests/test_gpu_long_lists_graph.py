"""GPU: long lists in parts under a captured graph.  The parts' counters and the
key image are state in the workspace that every pass has to start anew: each
replay, on other vertices and with eager work and synchronizations between
them, equals the eager result bit for bit."""
import numpy as np
import pytest

from tests.gpu_util import to_dev
from tests.test_gpu_long_lists import cluster

pytestmark = pytest.mark.gpu


def test_replays_equal_the_eager_result():
    import torch
    from paper_2405_02508_amd import mer
    H, W = 403, 517
    v_np, tri_np, attr_np, views = cluster(30000, H, W, (200, 100, 240, 150), 6.0)
    tri, attr = to_dev(tri_np), to_dev(attr_np)
    shift = np.random.default_rng(2).uniform(-20, 20, size=(5, 2)).astype(np.float32)
    inputs = [to_dev(v_np + np.array([dx, dy, 0], np.float32)) for dx, dy in shift]
    eager, ctx = mer.Context(views, device="cuda"), mer.Context(views, device="cuda")
    n = ctx.n_px
    new = lambda: (torch.empty(n, dtype=torch.int32, device="cuda"), torch.empty(n, device="cuda"),  # noqa: E731
                   torch.empty(n, 2, device="cuda"), torch.empty(n, 3, device="cuda"))
    v, out, ref = inputs[0].clone(), new(), new()
    run = lambda c, x, o: c.rasterize_interpolate(x, tri, o[0], attr, o[3], depth=o[1], bary=o[2])  # noqa: E731
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        run(ctx, v, out)
    torch.cuda.current_stream().wait_stream(s)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run(ctx, v, out)
    for x in inputs + inputs[:1]:
        v.copy_(x)
        for o in out:
            o.fill_(7)
        graph.replay()
        run(eager, x, ref)
        torch.cuda.synchronize()
        assert int(ctx.ws[ctx.plan.off_status:ctx.plan.off_status + 64].view(torch.int64)[3]) > 1
        for a, b in zip(out, ref):
            assert torch.equal(a, b)
        assert int((out[0] >= 0).sum()) > 1000 and float((out[3] * 2).sum()) > 0  # eager work between the replays
