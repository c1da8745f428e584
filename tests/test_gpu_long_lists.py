"""GPU: coarse tiles whose lists are longer than one workgroup's share,
against the CPU oracle bit for bit: the parts of a list are rasterized by
workgroups of their own and meet in memory, on each tile side, at the view's
ragged edge, over several views, for triangles listed by rank and by walking,
and where there is room for the parts of only a few of the tiles."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


def cluster(n, H, W, box, size, n_views=1, seed=11):
    """n triangles of up to ``size`` px with centres in box (x0, y0, x1, y1)."""
    rng = np.random.default_rng(seed + n)
    centre = rng.uniform(box[:2], box[2:], size=(n, 1, 2))
    xy = centre + rng.uniform(-size / 2, size / 2, size=(n, 3, 2))
    z = rng.uniform(1.0, 10.0, size=(n, 1, 1)) * (1.0 + 0.01 * rng.uniform(-1, 1, size=(n, 3, 1)))
    v = np.concatenate([xy, z], 2).reshape(-1, 3).astype(np.float32)
    tri = np.arange(3 * n, dtype=np.int32).reshape(n, 3)
    views = np.array([[0, 0, 0, i * H * W, 3 * n, n, H, W] for i in range(n_views)], np.int64)
    return v, tri, rng.uniform(size=(3 * n, 3)).astype(np.float32), views


CASES = {
    # name: (geometry, log2 of the tile side, every part finds room)
    "8px": (lambda: cluster(40000, 70, 90, (30, 20, 60, 45), 5.0), 3, True),
    "16px": (lambda: cluster(30000, 403, 517, (200, 100, 240, 150), 6.0), 4, True),
    "16px_views": (lambda: cluster(20000, 403, 517, (490, 380, 520, 410), 9.0, n_views=3), 4, True),
    "32px_edge": (lambda: cluster(30000, 1001, 1090, (1040, 960, 1095, 1005), 6.0), 5, True),
    "32px_walked": (lambda: cluster(14000, 1001, 1090, (500, 500, 520, 520), 400.0), 5, False),
    "8px_no_room": (lambda: cluster(30000, 64, 64, (0, 0, 64, 64), 200.0), 3, False),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_long_lists_match_the_oracle(name):
    import torch
    from paper_2405_02508_amd import mer
    make, ctl, room = CASES[name]
    v_np, tri_np, attr_np, views = make()
    n_t, H, W = (int(x) for x in views[0, 5:])
    say(f"[long lists] {name}: {n_t} triangles, {len(views)} x {W}x{H}")
    ctx = mer.Context(views, device="cuda", bin_cap=2000000)  # holds every list
    assert ctx.plan.ct_log2 == ctl
    v, tri, attr = to_dev(v_np), to_dev(tri_np), to_dev(attr_np)
    n = ctx.n_px
    tid = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    depth, bary = torch.full((n,), -7.0, device="cuda"), torch.full((n, 2), -7.0, device="cuda")
    out = torch.full((n, 3), -7.0, device="cuda")
    ref = oracle.rasterize(v_np, tri_np, H, W)
    ref_depth = oracle.resolve(v_np, tri_np, H, W, ref)[0]
    first = None
    for rep in range(3):
        ctx.rasterize_interpolate(v, tri, tid, attr, out, depth=depth, bary=bary)
        assert ctx.status()["overflow_tiles"] == 0
        parts = int(ctx.ws[ctx.plan.off_status:ctx.plan.off_status + 64].view(torch.int64)[3])
        room_for = (2 * n_t * len(views) // 1024 + 7) // 8 * 8
        assert parts > 1 and (parts <= room_for) == room, (parts, room_for)
        for i in range(len(views)):
            got = tid[i * H * W:(i + 1) * H * W].cpu().numpy()
            assert np.array_equal(got, ref), f"view {i}: tri_id differs at {int((got != ref).sum())} pixels"
            d = depth[i * H * W:(i + 1) * H * W].cpu().numpy()
            assert np.all(np.abs(d - ref_depth) <= 1e-5 * np.maximum(1, np.abs(ref_depth)))
        two = torch.empty_like(out)
        ctx.interpolate(attr, v, tri, tid, two, bary=bary)
        assert torch.equal(out, two)
        if first is None:
            first = [x.clone() for x in (tid, depth, bary, out)]
        assert all(torch.equal(a, b) for a, b in zip(first, (tid, depth, bary, out)))
