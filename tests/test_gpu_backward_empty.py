"""GPU: the backward sweep over tiles without a covered pixel, which it leaves
early, against the CPU oracle: views with nothing in them, with one triangle
whose border is the side of a 16 x 16 tile, and with a few.  Gradients within
1e-5 relative L2 per tensor (the parity bar); the loss, a sum of squares whose
terms carry one rounding each and whose partial sums over 64 pixels are
binary32, within 1e-5 relative; exact zeros where nothing is covered."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import rel_l2, say, to_dev

pytestmark = pytest.mark.gpu

TRIS = {
    "none": [],
    "one_tile": [[(16.5, 16.5), (31.5, 16.5), (16.5, 31.5)]],
    "to_the_side": [[(-40.0, 0.0), (16.0, 0.0), (-40.0, 90.0)], [(48.0, 3.0), (70.0, 3.0), (48.0, 40.0)]],
}


@pytest.mark.parametrize("loss", [True, False])
@pytest.mark.parametrize("name", list(TRIS))
@pytest.mark.parametrize("W,H", [(48, 48), (65, 35)])
def test_tiles_without_a_covered_pixel(W, H, name, loss):
    import torch
    from paper_2405_02508_amd import mer
    rng = np.random.default_rng(W)
    xy = np.array(TRIS[name] or [[(-9.0, -9.0), (-5.0, -9.0), (-9.0, -5.0)]]).reshape(-1, 2)
    v_np = np.concatenate([xy, rng.uniform(1.0, 2.0, size=(len(xy), 1))], 1).astype(np.float32)
    tri_np = np.arange(len(xy), dtype=np.int32).reshape(-1, 3)
    attr_np = rng.uniform(size=(len(xy), 3)).astype(np.float32)
    views = np.array([[0, 0, 0, 0, len(v_np), len(tri_np), H, W]], np.int64)
    say(f"[empty] {W}x{H} {name} loss {loss}")
    ctx = mer.Context(views, device="cuda")
    v, tri, attr = to_dev(v_np), to_dev(tri_np), to_dev(attr_np)
    tid = torch.empty(W * H, dtype=torch.int32, device="cuda")
    img = torch.empty(W * H, 3, device="cuda")
    ctx.rasterize_interpolate(v, tri, tid, attr, img)
    t_np = oracle.rasterize(v_np, tri_np, H, W)
    assert np.array_equal(tid.cpu().numpy(), t_np)
    target = rng.uniform(-1, 1, size=(W * H, 3)).astype(np.float32)
    im = img.cpu().numpy().astype(np.float64)
    g = 1.5 * (im - target)  # weight 0.75
    ref_v = oracle.edge_grad(v_np, tri_np, H, W, t_np, im, g)
    ref_a, ref_v = oracle.interpolate_bwd(attr_np, v_np, tri_np, H, W, t_np, g, False, g_v=ref_v)
    g_v, g_attr, total = torch.zeros_like(v), torch.zeros_like(attr), torch.zeros(1, device="cuda")
    ctx.backward_l2(v, tri, tid, attr, img, to_dev(target), g_attr, g_v, weight=0.75, loss=total if loss else None)
    if not (t_np >= 0).any():
        assert float(g_v.abs().max()) == 0.0 and float(g_attr.abs().max()) == 0.0
    else:
        assert rel_l2(g_v.cpu().numpy(), ref_v) <= 1e-5 and rel_l2(g_attr.cpu().numpy(), ref_a) <= 1e-5
    if loss:
        want = 0.75 * np.sum((im - target) ** 2)
        assert abs(total.item() - want) <= 1e-5 * want
