"""GPU: the backward sweep for attribute rows around and beyond the eight
channels its vertex table takes at once, and the loss summed in the sweep,
against the CPU oracle.  Gradients within 1e-5 relative L2 per tensor (the
parity bar); the loss, a sum of squares whose terms carry one rounding each
and whose partial sums over 64 pixels are binary32, within 1e-5 relative."""
import numpy as np
import pytest

import oracle
from paper_2405_02508_amd import scenes
from tests.gpu_util import rel_l2, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("append_z", [False, True])
@pytest.mark.parametrize("C", [1, 8, 9, 12, 13, 16, 17, 63])
def test_wide_attribute_rows(C, append_z):
    import torch
    from paper_2405_02508_amd import mer
    s = scenes.make_config(2, small=True)
    vw = s.view(0)
    H, W = vw["H"], vw["W"]
    rng = np.random.default_rng(C)
    attr_np = rng.uniform(-1, 1, size=(s.attr.shape[0], C)).astype(np.float32)
    Ce = C + int(append_z)
    say(f"[wide] {C} channels, append_z {append_z}")
    ctx = mer.Context(s.views, device="cuda")
    v, tri, attr = to_dev(s.v), to_dev(s.tri), to_dev(attr_np)
    n = ctx.n_px
    tid = torch.empty(n, dtype=torch.int32, device="cuda")
    img = torch.empty(n, Ce, device="cuda")
    ctx.rasterize_interpolate(v, tri, tid, attr, img, append_z=append_z)
    t_np = oracle.rasterize(s.v, s.tri, H, W)
    assert np.array_equal(tid.cpu().numpy(), t_np)
    target = rng.uniform(-1, 1, size=(n, Ce)).astype(np.float32)
    im = img.cpu().numpy().astype(np.float64)
    g = 1.5 * (im - target)  # weight 0.75
    ref_v = oracle.edge_grad(s.v, s.tri, H, W, t_np, im, g)
    ref_a, ref_v = oracle.interpolate_bwd(attr_np, s.v, s.tri, H, W, t_np, g, append_z, g_v=ref_v)
    ref_loss = 0.75 * np.sum((im - target) ** 2)
    g_v, g_attr, loss = torch.zeros_like(v), torch.zeros_like(attr), torch.zeros(1, device="cuda")
    ctx.backward_l2(v, tri, tid, attr, img, to_dev(target), g_attr, g_v, weight=0.75, loss=loss, append_z=append_z)
    assert rel_l2(g_v.cpu().numpy(), ref_v) <= 1e-5 and rel_l2(g_attr.cpu().numpy(), ref_a) <= 1e-5
    assert abs(loss.item() - ref_loss) <= 1e-5 * ref_loss
    # the same from a given dL/d(image), and the interpolation adjoint alone
    g_v.zero_(), g_attr.zero_()
    gd = to_dev(g.astype(np.float32))
    ctx.backward(v, tri, tid, attr, img, gd, g_attr, g_v, append_z=append_z)
    assert rel_l2(g_v.cpu().numpy(), ref_v) <= 1e-5 and rel_l2(g_attr.cpu().numpy(), ref_a) <= 1e-5
    g_attr.zero_()
    ctx.interpolate_bwd(attr, v, tri, tid, gd, g_attr, None, append_z=append_z)
    assert rel_l2(g_attr.cpu().numpy(), ref_a) <= 1e-5
