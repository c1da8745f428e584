"""GPU: the coverage channel written with the interpolated image is, bit for
bit, the image without it and the index image's coverage beside it, for row
widths of every store (four, three, single), with and without z, on both
rasterizers and on tiles of background."""
import numpy as np
import pytest

from paper_2405_02508_amd import scenes
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("small_px", [0, -1])
@pytest.mark.parametrize("C,append_z", [(1, False), (1, True), (2, False), (3, False), (6, True), (7, False),
                                        (11, True), (63, True), (64, False)])
def test_mask_channel_is_the_coverage(C, append_z, small_px):
    import torch
    from paper_2405_02508_amd import mer
    s = scenes.scattered_triangles(C, 40, 75, 133, 25.0)
    say(f"[mask] {C} channels, z {append_z}, small_px {small_px}")
    ctx = mer.Context(s.views, device="cuda", small_px=small_px)
    attr = to_dev(np.random.default_rng(C).uniform(-1, 1, size=(s.v.shape[0], C)).astype(np.float32))
    v, tri, n = to_dev(s.v), to_dev(s.tri), ctx.n_px
    for bary in (None, torch.empty(n, 2, device="cuda")):
        tid = torch.empty(n, dtype=torch.int32, device="cuda")
        out, img = torch.empty(n, C + append_z, device="cuda"), torch.full((n, C + append_z + 1), -7.0, device="cuda")
        ctx.rasterize_interpolate(v, tri, tid, attr, out, bary=bary, append_z=append_z)
        want = torch.cat([out, (tid >= 0).float()[:, None]], 1)
        ctx.rasterize_interpolate(v, tri, tid, attr, img, bary=bary, append_z=append_z, mask=True)
        assert 0 < int((tid >= 0).sum()) < n
        assert torch.equal(img.view(torch.int32), want.view(torch.int32))
