"""GPU: attribute gradients of channels whose dL/d(image) differ by many
decades, against the CPU oracle, channel by channel.

From the ninth channel on every partial sum of a channel is binary32 (each
rounded by at most 2^-24 of itself), so a channel is as accurate whatever its
neighbours hold: within 1e-5 relative L2 per channel, the parity bar of a
whole tensor, with the scales spread over 36 decades."""
import numpy as np
import pytest

import oracle
from paper_2405_02508_amd import scenes
from tests.gpu_util import rel_l2, say, to_dev

pytestmark = pytest.mark.gpu

SCALES = (1.0, 1e-3, 2.0 ** -24, 1e6, 1e-18, 1e18, 1e-9, 1.0)


@pytest.mark.parametrize("call", ["interpolate_bwd", "backward", "backward_l2"])
@pytest.mark.parametrize("C", [9, 12, 16, 23])
def test_channels_of_unlike_scale(C, call):
    import torch
    from paper_2405_02508_amd import mer
    s = scenes.make_config(2, small=True)
    vw = s.view(0)
    H, W = vw["H"], vw["W"]
    rng = np.random.default_rng(100 + C)
    attr_np = rng.uniform(-1, 1, size=(s.attr.shape[0], C)).astype(np.float32)
    scale = np.array([SCALES[c % len(SCALES)] for c in range(C)])
    say(f"[scales] {C} channels, {call}")
    ctx = mer.Context(s.views, device="cuda")
    v, tri, attr = to_dev(s.v), to_dev(s.tri), to_dev(attr_np)
    n = ctx.n_px
    tid = torch.empty(n, dtype=torch.int32, device="cuda")
    img = torch.empty(n, C, device="cuda")
    ctx.rasterize_interpolate(v, tri, tid, attr, img)
    t_np = oracle.rasterize(s.v, s.tri, H, W)
    assert np.array_equal(tid.cpu().numpy(), t_np)
    g = (rng.uniform(-1, 1, size=(n, C)) * scale).astype(np.float32)
    g_attr = torch.zeros_like(attr)
    if call == "interpolate_bwd":
        ctx.interpolate_bwd(attr, v, tri, tid, to_dev(g), g_attr, None)
    elif call == "backward":
        ctx.backward(v, tri, tid, attr, img, to_dev(g), g_attr, torch.zeros_like(v))
    else:  # dL/d(image) = 2 (img - target), with the image scaled as its gradient
        img = to_dev(g)
        target = torch.zeros_like(img)
        g = 2.0 * g
        ctx.backward_l2(v, tri, tid, attr, img, target, g_attr, torch.zeros_like(v), weight=1.0)
    ref, _ = oracle.interpolate_bwd(attr_np, s.v, s.tri, H, W, t_np, g.astype(np.float64), False)
    got = g_attr.cpu().numpy()
    for c in range(8, C):
        assert rel_l2(got[:, c], ref[:, c]) <= 1e-5, f"channel {c} of scale {scale[c]:g}"
