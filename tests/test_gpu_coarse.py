"""GPU: the coarse-tile rasterizer at the edges of its rules, against the CPU
oracle: index image bit for bit, depth within the parity bar, the integrity
counts of the lists zero, and the one-pass interpolation bit-identical to
rasterizing then interpolating.

The plans cover the three tile sides, the list-free launch of a small view
and the lists, tiles with more candidates than one chunk, triangles over one,
four, a few and many tiles, lists that overflow the pool, and triangles whose
extent is the largest of the 16-bit records or one step more."""
import numpy as np
import pytest

import oracle
from paper_2405_02508_amd import scenes
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


def extent_scene(n, W, H):
    """n triangles whose x or y extent is 32766 .. 32769 steps of 1/256 px,
    placed so that their boxes begin at every offset from a tile's edge."""
    rng = np.random.default_rng(5)
    ext = rng.integers(32766, 32770, size=(n, 2))
    ext[::2, 1] = rng.integers(256, 20000, size=ext[::2, 1].shape)
    o = np.stack([rng.integers(0, 256 * (W - 64), size=n), rng.integers(0, 256 * (H - 64), size=n)], 1)
    u = rng.integers(0, 3, size=(n, 2))  # which vertex sits inside the box, per axis
    xy = np.zeros((n, 3, 2), np.int64)
    for a in (0, 1):
        mid = (rng.uniform(size=n) * ext[:, a]).astype(np.int64)
        for k in range(3):
            xy[:, k, a] = o[:, a] + np.where(u[:, a] == k, mid, np.where((u[:, a] + 1) % 3 == k, 0, ext[:, a]))
    z = rng.uniform(1.0, 10.0, size=(n, 3, 1))
    v = np.concatenate([xy / 256.0, z], 2).reshape(-1, 3).astype(np.float32)
    tri = np.arange(3 * n, dtype=np.int32).reshape(n, 3)
    attr = rng.uniform(size=(3 * n, 5)).astype(np.float32)
    views = np.array([[0, 0, 0, 0, 3 * n, n, H, W]], np.int64)
    return v, tri, attr, views


def scattered(n, W, H, size, n_views=1):
    s = scenes.scattered_triangles(n + W, n, H, W, size)
    views = np.repeat(s.views, n_views, 0)
    views[:, 3] = np.arange(n_views) * H * W  # the same geometry in every view
    return s.v, s.tri, s.attr, views


CASES = {
    # name: (geometry, bin_cap, log2 of the tile side)
    "direct_one_chunk": (lambda: scattered(256, 61, 67, 30.0), 0, 4),
    "direct_two_chunks": (lambda: scattered(257, 64, 64, 5.0), 0, 4),
    "lists_8px": (lambda: scattered(13000, 120, 90, 9.0), 0, 3),
    "lists_16px": (lambda: scattered(6000, 400, 300, 30.0), 0, 4),
    "lists_16px_views": (lambda: scattered(900, 201, 99, 50.0, n_views=3), 0, 4),
    "lists_32px_large": (lambda: scattered(1500, 1090, 1001, 300.0), 0, 5),
    "lists_32px_small": (lambda: scattered(60000, 1090, 1001, 6.0), 0, 5),
    "overflow_16px": (lambda: scattered(3000, 400, 300, 30.0), 300, 4),
    "overflow_32px": (lambda: scattered(800, 1090, 1001, 200.0), 1000, 5),
    "extents_16px": (lambda: extent_scene(600, 500, 420), 0, 4),
    "extents_32px": (lambda: extent_scene(900, 1090, 1001), 0, 5),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_coarse_tiles_match_the_oracle(name):
    import torch
    from paper_2405_02508_amd import mer
    make, cap, ctl = CASES[name]
    v_np, tri_np, attr_np, views = make()
    n_v, n_t, H, W = (int(x) for x in views[0, 4:])
    say(f"[coarse] {name}: {n_t} triangles, {len(views)} x {W}x{H}")
    ctx = mer.Context(views, device="cuda", bin_cap=cap)
    assert ctx.plan.ct_log2 == ctl
    v, tri, attr = to_dev(v_np), to_dev(tri_np), to_dev(attr_np)
    n = ctx.n_px
    tid = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    depth, bary = torch.full((n,), -7.0, device="cuda"), torch.full((n, 2), -7.0, device="cuda")
    both = torch.full((n, attr.shape[1] + 1), -7.0, device="cuda")
    two = torch.full_like(both, -5.0)
    ctx.rasterize_interpolate(v, tri, tid, attr, both, depth=depth, bary=bary, append_z=True)
    st = ctx.status()  # raises on a nonzero integrity count
    assert (st["overflow_tiles"] > 0) == (cap > 0)
    ref = oracle.rasterize(v_np, tri_np, H, W)
    ref_depth = oracle.resolve(v_np, tri_np, H, W, ref)[0]
    for i in range(len(views)):
        got = tid[i * H * W:(i + 1) * H * W].cpu().numpy()
        assert np.array_equal(got, ref), f"view {i}: tri_id differs at {int((got != ref).sum())} pixels"
        d = depth[i * H * W:(i + 1) * H * W].cpu().numpy()
        assert np.all(np.abs(d - ref_depth) <= 1e-5 * np.maximum(1, np.abs(ref_depth)))
    tid2 = torch.empty_like(tid)
    ctx.rasterize(v, tri, tid2, None, bary)
    ctx.interpolate(attr, v, tri, tid2, two, bary=bary, append_z=True)
    assert torch.equal(tid, tid2) and torch.equal(both, two)
    ctx.interpolate(attr, v, tri, tid2, two, bary=None, append_z=True)
    assert torch.equal(both, two)
