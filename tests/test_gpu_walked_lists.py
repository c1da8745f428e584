"""GPU: coarse lists of many triangles that each cover more tiles than the
count pass takes (their tiles are walked), against the CPU oracle bit for bit,
and against the time of per-tile lists of the same scene: the coarse lists are
the default, so they may not be the slower ones.  They were once, by half
(one triangle a workgroup, and a counter read again beside its own atomics);
they take 0.5 to 0.7 of the time, so 1.1 leaves room for a busy machine."""
import numpy as np
import pytest

import oracle
from paper_2405_02508_amd import scenes
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


def _time(fn, reps=10):
    import torch
    best = float("inf")
    for _ in range(4):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(reps):
            fn()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / reps)
    return best


@pytest.mark.parametrize("n_t,size,side", [(100000, 40.0, 256), (200000, 60.0, 1024), (500, 60.0, 300), (5, 400.0, 300)])
def test_walked_lists(n_t, size, side):
    import torch
    from paper_2405_02508_amd import mer
    s = scenes.scattered_triangles(3, n_t, side, side, size)
    say(f"[walked] {n_t} triangles of up to {size} px, {side} x {side}")
    v, tri = to_dev(s.v), to_dev(s.tri)
    ref = oracle.rasterize(s.v, s.tri, side, side)
    ms = {}
    for small_px in (0, -1):
        ctx = mer.Context(s.views, device="cuda", small_px=small_px)
        tid = torch.full((ctx.n_px,), -7, dtype=torch.int32, device="cuda")
        ctx.rasterize(v, tri, tid)
        assert ctx.status()["overflow_tiles"] == 0
        assert np.array_equal(tid.cpu().numpy(), ref)
        ms[small_px] = _time(lambda: ctx.rasterize(v, tri, tid))
    say(f"    {ms[0]:.3f} ms, per-tile lists {ms[-1]:.3f} ms")
    if n_t >= 100000:
        assert ms[0] <= 1.1 * ms[-1]
