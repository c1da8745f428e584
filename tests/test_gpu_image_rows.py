"""GPU: the image rows the rasterizer writes, by lane or by way of LDS, are bit
for bit the interpolation module's for the same pixels: every width around the
rule's lines, on each tile side, with views whose right and lower tiles are cut
and rows that begin at every alignment."""
import numpy as np
import pytest

from paper_2405_02508_amd import scenes
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu

VIEWS = {"8px": (13000, 91, 121, 1, 3), "16px": (300, 99, 201, 3, 4), "32px": (1500, 1001, 1090, 2, 5)}


@pytest.mark.parametrize("C", [1, 2, 4, 5, 6, 7, 8, 9, 11, 13, 15, 16, 17])
@pytest.mark.parametrize("name", list(VIEWS))
def test_rows_match_the_interpolation_module(name, C):
    import torch
    from paper_2405_02508_amd import mer
    n_tri, H, W, n_views, ctl = VIEWS[name]
    s = scenes.scattered_triangles(C, n_tri, H, W, 9.0 if ctl == 3 else 40.0)
    views = np.repeat(s.views, n_views, 0)
    views[:, 3] = np.arange(n_views) * H * W
    say(f"[rows] {name}, {C} channels")
    ctx = mer.Context(views, device="cuda")
    assert ctx.plan.ct_log2 == ctl
    attr = to_dev(np.random.default_rng(C).uniform(-1, 1, size=(s.v.shape[0], C)).astype(np.float32))
    v, tri, n = to_dev(s.v), to_dev(s.tri), ctx.n_px
    tid, bary = torch.empty(n, dtype=torch.int32, device="cuda"), torch.empty(n, 2, device="cuda")
    for shift in (0, 1):  # a base that no vector store takes
        buf = torch.full((n * C + shift,), -7.0, device="cuda")
        img, want = buf[shift:].view(n, C), torch.empty(n, C, device="cuda")
        ctx.rasterize_interpolate(v, tri, tid, attr, img, bary=bary)
        ctx.interpolate(attr, v, tri, tid, want, bary=bary)
        assert torch.equal(img.contiguous().view(torch.int32), want.view(torch.int32))
        assert shift == 0 or float(buf[0]) == -7.0
