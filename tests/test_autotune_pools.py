"""The autotuner's measuring and its cache, with the device calls replaced: a
cached pool is used only where it holds the lists it was measured for, and each
candidate is a rasterizer of its own.  No GPU needed."""
import json

import numpy as np
import pytest
import torch

from paper_2405_02508_amd import autotune, mer


def _view(H, W, n_t, n=1):
    return np.array([[0, 0, 0, i * H * W, 3, n_t, H, W] for i in range(n)], np.int64)


class _Event:
    def __init__(self, **kw):
        pass

    def record(self, *a):
        pass

    def elapsed_time(self, other):
        return 1.0


@pytest.fixture
def measured(monkeypatch):
    """Plans measured, and the entries each is to report."""
    made = []

    class Context:
        entries = 1000

        def __init__(self, views, device, tile, small_px, big_tiles, bin_cap=0):
            self.plan = mer.plan_init(views, tile, bin_cap, small_px, big_tiles)
            made.append((tile, small_px, big_tiles, bin_cap))

        def rasterize(self, *a):
            pass

        def status(self):
            return {"entries": Context.entries}

    monkeypatch.setattr(autotune.mer, "Context", Context)
    for name, f in (("current_stream", lambda: None), ("synchronize", lambda: None), ("empty_cache", lambda: None),
                    ("Event", _Event)):
        monkeypatch.setattr(torch.cuda, name, f)
    made_by = lambda n: setattr(Context, "entries", n)  # noqa: E731
    return made, made_by


def test_a_plan_without_lists_leaves_no_pool_to_one_with_lists(tmp_path, measured):
    made, report = measured
    path = str(tmp_path / "tune.json")
    small, listed = _view(64, 64, 2000), _view(64, 64, 2800)
    assert autotune.shape_class(small) == autotune.shape_class(listed)
    report(0)  # what the rasterizer without lists reports
    assert autotune.tune(small, None, None, device="cpu", cache_path=path)["bin_cap"] == 0
    n = len(made)
    got = autotune.tune(listed, None, None, device="cpu", cache_path=path)
    assert got["cached"] and len(made) == n
    assert got["bin_cap"] == 0  # the default, which is sized from the plan


def test_a_pool_belongs_to_the_side_of_its_tiles(tmp_path, measured):
    made, report = measured
    path = str(tmp_path / "tune.json")
    wide, fine = _view(1024, 1024, 100000), _view(990, 990, 100000)
    assert autotune.shape_class(wide) == autotune.shape_class(fine)
    assert mer.plan_init(wide).ct_log2 != mer.plan_init(fine).ct_log2
    report(50000)
    autotune.tune(wide, None, None, device="cpu", cache_path=path)
    n = len(made)
    assert autotune.tune(wide, None, None, device="cpu", cache_path=path)["cached"] and len(made) == n
    assert not autotune.tune(fine, None, None, device="cpu", cache_path=path)["cached"] and len(made) > n
    n = len(made)  # each is kept beside the other
    for V in (wide, fine):
        assert autotune.tune(V, None, None, device="cpu", cache_path=path)["cached"]
    assert len(made) == n


def test_a_pool_grows_with_what_it_is_used_for(tmp_path, measured):
    made, report = measured
    path = str(tmp_path / "tune.json")
    V = _view(800, 800, 80000)
    report(100000)
    cap = autotune.tune(V, None, None, device="cpu", cache_path=path)["bin_cap"]
    assert cap == 129096  # a quarter and 4096 more than the entries
    more = _view(800, 800, 90000)
    assert autotune.shape_class(V) == autotune.shape_class(more)
    assert autotune.tune(more, None, None, device="cpu", cache_path=path)["bin_cap"] == int(cap * 90000 / 80000)
    fewer = _view(790, 800, 70000)
    assert autotune.shape_class(V) == autotune.shape_class(fewer)
    assert autotune.tune(fewer, None, None, device="cpu", cache_path=path)["bin_cap"] == cap


def test_an_entry_of_a_class_alone_keeps_the_default_pool(tmp_path):
    V = _view(64, 64, 3000)
    path = tmp_path / "tune.json"
    entry = {"tile": [8, 8], "small_px": 16, "big_tiles": 16, "bin_cap": 4096, "entries": 0, "ms": 1.0, "lists": "coarse"}
    path.write_text(json.dumps({autotune.shape_class(V): entry}))
    got = autotune.tune(V, None, None, cache_path=str(path))
    assert got["cached"] and got["bin_cap"] == 0 and got["tile"] == (8, 8)


def test_no_rasterizer_is_measured_twice(tmp_path, measured):
    made, report = measured
    V = _view(300, 300, 5000)
    out = autotune.tune(V, None, None, device="cpu", cache_path=str(tmp_path / "t.json"))
    coarse = [r for r in out["table"] if r["small_px"] >= 0]
    assert len(coarse) == 1 and len(out["table"]) == len(autotune.CANDIDATES) == 4
    same = ((8, 8, 16, 16), (16, 16, 256, -1), (32, 8, 64, 4), (8, 8, -1, 16), (8, 8, -3, 16))
    out = autotune.tune(V, None, None, device="cpu", candidates=same, cache_path=None)
    assert [(tuple(r["tile"]), r["small_px"]) for r in out["table"]] == [((8, 8), 16), ((8, 8), -1)]
