"""A cached tuning is used only for the lists its bin pool was measured for."""
import json

import numpy as np
import pytest

from paper_2405_02508_amd import autotune


class Measured(Exception):
    pass


@pytest.mark.parametrize("small_px,lists,used", [(-1, None, True), (-1, "tile", True), (0, None, False),
                                                 (256, None, False), (256, "coarse", True), (16, "tile", False)])
def test_cached_pool_belongs_to_its_lists(tmp_path, monkeypatch, small_px, lists, used):
    V = np.array([[0, 0, 0, 0, 3, 1000, 64, 64]], np.int64)
    entry = {"tile": [8, 8], "small_px": small_px, "big_tiles": 16, "bin_cap": 10, "entries": 8, "ms": 1.0}
    if lists:
        entry["lists"] = lists
    path = tmp_path / "tune.json"
    path.write_text(json.dumps({autotune.shape_class(V): entry}))

    def measure(*a, **k):
        raise Measured

    monkeypatch.setattr(autotune.mer, "plan_init", measure)
    if used:
        assert autotune.tune(V, None, None, cache_path=str(path))["cached"]
    else:
        with pytest.raises(Measured):
            autotune.tune(V, None, None, cache_path=str(path))
