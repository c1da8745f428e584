"""Autotuner for the rasterizer (lists of coarse tiles, or per-tile lists with
their tile shape and large-triangle limit) and its bin pool.

None of these change the results (the visibility rule is order-independent
and the overflow path is exact); they only change speed and workspace size.
For a view table and its geometry the tuner:
  1. runs mer_rasterize once per candidate and reads the number of
     triangle-tile entries from mer_status, so the bin pool can be sized to
     what the workload needs (plus a margin) instead of a worst case;
  2. times mer_rasterize for each candidate with HIP events on the current
     stream and keeps the fastest.
Choices are cached in a JSON file keyed by a shape class (view count,
pixel and triangle counts rounded to powers of two) and the side of the coarse
tiles, since a pool belongs to its lists (one too small for them is exact but
slow): within a class it grows with the pixels and triangles it is used for.  A
plan that needs no lists (a small view of few triangles) measures no entries:
it keeps the default pool, bin_cap 0.  Entries of a class alone are from before
the side was part of the key: those of per-tile lists hold, those of coarse
tiles get the default pool, and those from before there were coarse tiles, when
triangles of few pixels took no entries, are measured anew.
"""
from __future__ import annotations

import json
import math
import os

import numpy as np

from . import mer

CANDIDATES = (
    # (tile_w, tile_h, small_px, big_tiles): the coarse tiles, whatever the
    # other three are, and the per-tile lists (small_px < 0)
    (8, 8, 16, 16),
    (8, 8, -1, 16), (8, 8, -1, -1), (16, 16, -1, 16),
)
DEFAULT_CACHE = os.path.join(os.path.expanduser("~"), ".cache", "mer_autotune.json")


def shape_class(views_i64) -> str:
    V = np.asarray(views_i64, np.int64)
    px = int((V[:, 6] * V[:, 7]).sum())
    tris = int(V[:, 5].sum())
    b = lambda x: int(round(math.log2(max(x, 1))))  # noqa: E731
    return f"v2-v{V.shape[0]}-px2^{b(px)}-t2^{b(tris)}"


def _load(path):
    try:
        with open(path) as f:
            return json.load(f)
    except (OSError, ValueError):
        return {}


def _totals(views_i64):
    V = np.asarray(views_i64, np.int64)
    return int((V[:, 6] * V[:, 7]).sum()), int(V[:, 5].sum())


def _reuse(data, views_i64):
    """The cached choice for these views (without its measurements), or None."""
    key = shape_class(views_i64)
    hit = data.get(key)  # of a class alone
    if hit and hit.get("small_px", 0) < 0:
        return dict(hit)
    if hit and hit.get("lists") == "coarse":
        return dict(hit, bin_cap=0)
    hit = data.get(_side_key(views_i64))
    if not hit:
        return None
    px, tris = _totals(views_i64)
    grow = max(1.0, px / hit["px"]) * max(1.0, tris / hit["tris"])
    return dict(hit, bin_cap=min(int(hit["bin_cap"] * grow), 2**31 - 2))


def _side_key(views_i64):
    return f"{shape_class(views_i64)}-c{1 << mer.plan_init(views_i64).ct_log2}"


def tune(views_i64, v, tri, device="cuda", candidates=CANDIDATES, reps=3, cache_path=DEFAULT_CACHE,
         use_cache=True, log=None):
    """Return dict(tile=(w, h), small_px=int, big_tiles=int, bin_cap=int, ms=float, table=[...])."""
    import torch
    key = shape_class(views_i64)
    if use_cache and cache_path:
        hit = _reuse(_load(cache_path), views_i64)
        if hit:
            return dict(hit, tile=tuple(hit["tile"]), cached=True)
    n_px = int(mer.plan_init(views_i64).total_px)
    tid = torch.empty(n_px, dtype=torch.int32, device=device)
    depth = torch.empty(n_px, dtype=torch.float32, device=device)
    bary = torch.empty(n_px, 2, dtype=torch.float32, device=device)
    stream = torch.cuda.current_stream()
    table = []
    best = None
    seen = set()
    for (tw, th, sp, bt) in candidates:
        runs = (tw, th, bt) if sp < 0 else "coarse"  # what the candidate makes a plan of
        if runs in seen:
            continue
        seen.add(runs)
        ctx = mer.Context(views_i64, device=device, tile=(tw, th), small_px=sp, big_tiles=bt)
        ctx.rasterize(v, tri, tid, depth, bary)
        st = ctx.status()
        cap = int(st["entries"] * 1.25) + 4096 if st["entries"] else 0
        del ctx
        ctx = mer.Context(views_i64, device=device, tile=(tw, th), small_px=sp, big_tiles=bt, bin_cap=cap)
        ctx.rasterize(v, tri, tid, depth, bary)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        e0.record(stream)
        for _ in range(reps):
            ctx.rasterize(v, tri, tid, depth, bary)
        e1.record(stream)
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1) / reps
        row = dict(tile=(tw, th), small_px=sp, big_tiles=bt, bin_cap=cap, entries=int(st["entries"]), ms=round(ms, 4))
        table.append(row)
        if log:
            log(f"[autotune] {row}")
        if best is None or ms < best["ms"]:
            best = row
        del ctx
        torch.cuda.empty_cache()
    out = dict(best, table=table, key=key, cached=False)
    if cache_path:
        data = _load(cache_path)
        px, tris = _totals(views_i64)
        data[_side_key(views_i64)] = dict({k: out[k] for k in ("tile", "small_px", "big_tiles", "bin_cap", "entries", "ms")},
                                          px=px, tris=max(tris, 1))
        os.makedirs(os.path.dirname(cache_path), exist_ok=True)
        tmp = cache_path + ".tmp"
        with open(tmp, "w") as f:
            json.dump(data, f, indent=1)
        os.replace(tmp, cache_path)
    return out
