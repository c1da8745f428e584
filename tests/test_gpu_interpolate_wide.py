"""GPU: the interpolation module for rows of every write it has (staged close
together, staged apart and written 16 bytes a lane), on images whose last
workgroup is partly filled and on views with a gap between them, bit for bit
what the rasterizer's own resolve writes for the same pixels."""
import numpy as np
import pytest

from paper_2405_02508_amd import scenes
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stored", [True, False])
@pytest.mark.parametrize("gap", [0, 37])
@pytest.mark.parametrize("C,append_z", [(1, False), (8, False), (11, True), (12, False), (16, False), (16, True),
                                        (31, True), (33, False), (36, False), (63, True), (64, False)])
def test_interpolated_rows(C, append_z, gap, stored):
    import torch
    from paper_2405_02508_amd import mer
    s = scenes.scattered_triangles(C, 60, 71, 93, 30.0)
    views = np.repeat(s.views, 2, 0)
    views[1, 3] = 71 * 93 + gap
    say(f"[interp] {C} channels, z {append_z}, gap {gap}, stored {stored}")
    ctx = mer.Context(views, device="cuda")
    attr = to_dev(np.random.default_rng(C).uniform(-1, 1, size=(s.v.shape[0], C)).astype(np.float32))
    v, tri, n = to_dev(s.v), to_dev(s.tri), ctx.n_px
    tid = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    bary = torch.empty(n, 2, device="cuda")
    want, got = torch.full((n, C + append_z), -7.0, device="cuda"), torch.full((n, C + append_z), -7.0, device="cuda")
    ctx.rasterize_interpolate(v, tri, tid, attr, want, bary=bary, append_z=append_z)
    ctx.interpolate(attr, v, tri, tid, got, bary=bary if stored else None, append_z=append_z)
    assert torch.equal(got.view(torch.int32), want.view(torch.int32))
