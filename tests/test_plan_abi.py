"""mer_plan lies in its caller's memory and mer_plan_init fills it: a caller
compiled against a header of version 1 has 232 bytes of it, whatever the
library adds.  No GPU needed."""
import ctypes
import os

import numpy as np
import pytest

from paper_2405_02508_amd import mer

V1_BYTES = 232


@pytest.fixture(scope="module")
def L():
    if not os.path.exists(mer.LIB_PATH):
        from paper_2405_02508_amd import build
        build.build()
    return mer.lib()


@pytest.mark.parametrize("small_px", [0, 64, -1])
@pytest.mark.parametrize("H,W,n_t", [(64, 64, 320), (1100, 1300, 70000)])
def test_plan_init_writes_nothing_past_a_version_1_plan(L, H, W, n_t, small_px):
    assert L.mer_version() == 1
    buf = (ctypes.c_ubyte * (V1_BYTES + 64))(*([0xA5] * (V1_BYTES + 64)))
    views = mer.views_struct(np.array([[0, 0, 0, 0, 3, n_t, H, W]], np.int64))
    tun = mer.Tuning(8, 8, 0, small_px, 0)
    plan = ctypes.cast(buf, ctypes.POINTER(mer.Plan))
    assert L.mer_plan_init(views, 1, ctypes.byref(tun), plan) == 0
    assert plan.contents.total_tris == n_t and plan.contents.ws_bytes > 0
    assert set(buf[V1_BYTES:]) == {0xA5}
    assert ctypes.sizeof(mer.Plan) == V1_BYTES
