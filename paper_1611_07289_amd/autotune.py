"""Autotuner for the launch shapes of a plan's two PSF kernels.

Forward pass: the global-memory walk with its XCD granule (how many
consecutive work items one XCD takes at a time: of 256 blocks of 2 x 2 samples
where samples share their walk, else of 1024 samples), or LDS-staged tiles of
tile_w x tile_h pixels per workgroup.  Adjoint: the XCD granule of its
brick list.  Every candidate is applied (pvr_plan_set_tiles,
pvr_plan_set_granules) and its kernel timed with HIP events over a few
repetitions (median); the fastest of each kernel is kept and remembered in a
JSON cache keyed by the workload signature (problem sizes, patch sizes,
stack frames, PSF and cutoff), so later plans of the same workload skip the
search.  Granules change no result (every output keeps its summation order);
tiles walk every sample by itself and agree with walks that samples share to
the FP32 rounding of a sample.
"""
from __future__ import annotations

import hashlib
import json
import os
from typing import Dict, Optional

import numpy as np

# forward candidates: ("walk", granule) or ("tiles", tile_w, tile_h)
FORWARD = [("walk", 1), ("walk", 2), ("walk", 4), ("walk", 16),
           ("tiles", 16, 16), ("tiles", 32, 8), ("tiles", 8, 32), ("tiles", 64, 4)]
# adjoint candidates: XCD granules of the brick list
ADJOINT = [1, 4, 16, 32, 64, 256]
CACHE = os.environ.get("PVR_AUTOTUNE_CACHE",
                       os.path.join(os.path.expanduser("~"), ".cache", "pvr_mi355x",
                                    "autotune.json"))


def signature(plan) -> str:
    """The cache key; its prefix changes with the kernels that were timed."""
    h = hashlib.sha1()
    h.update(np.asarray([plan.N, plan.M, plan.V, plan.P], np.int64).tobytes())
    h.update(bytes(plan._g))
    h.update(bytes(plan._s))
    h.update(np.asarray([plan.psf, plan.cutoff_k], np.float64).tobytes())
    wh = np.asarray([(p.w, p.h) for p in plan._p], np.int32)
    h.update(np.unique(wh, axis=0).tobytes())
    return "v3-" + h.hexdigest()[:16]


def _load_cache(path: str) -> Dict:
    try:
        with open(path) as f:
            return json.load(f)
    except (OSError, ValueError):
        return {}


def _save_cache(path: str, data: Dict) -> None:
    try:
        os.makedirs(os.path.dirname(path), exist_ok=True)
        tmp = path + ".tmp"
        with open(tmp, "w") as f:
            json.dump(data, f, indent=1, sort_keys=True)
        os.replace(tmp, path)
    except OSError:
        pass


def _name(c) -> str:
    return f"walk/g{c[1]}" if c[0] == "walk" else f"tiles/{c[1]}x{c[2]}"


def _apply(plan, fwd, bp_granule):
    if fwd[0] == "walk":
        plan.set_tiles(0, 0)
        plan.set_granules(fwd[1], bp_granule)
    else:
        plan.set_granules(1, bp_granule)
        plan.set_tiles(fwd[1], fwd[2])


def _median_ms(fn, reps):
    import torch
    fn()  # warm
    evs = [torch.cuda.Event(enable_timing=True) for _ in range(reps + 1)]
    evs[0].record()
    for r in range(reps):
        fn()
        evs[r + 1].record()
    torch.cuda.synchronize()
    return sorted(evs[r].elapsed_time(evs[r + 1]) for r in range(reps))[reps // 2]


def tune(plan, X, y, reps: int = 3, cache: Optional[str] = CACHE, forward=FORWARD,
         adjoint=ADJOINT) -> Dict:
    """Pick and apply the fastest forward launch shape and adjoint granule
    for this plan (which must be built).  Returns {"forward": name,
    "adjoint_granule": g, "forward_ms": {...}, "adjoint_ms": {...}}."""
    import torch
    key = signature(plan)
    db = _load_cache(cache) if cache else {}
    if key in db:
        r = db[key]
        fwd = next(c for c in forward if _name(c) == r["forward"])
        _apply(plan, fwd, r["adjoint_granule"])
        return r
    dev = X.device
    e = torch.empty(plan.N, dtype=torch.float32, device=dev)
    p = torch.ones(plan.N, dtype=torch.float32, device=dev)
    W = torch.ones(plan.M, dtype=torch.float32, device=dev)
    num = torch.empty(plan.V, dtype=torch.float32, device=dev)
    den = torch.empty_like(num)
    fwd_ms = {}
    for c in forward:
        _apply(plan, c, 64)
        fwd_ms[_name(c)] = _median_ms(lambda: plan.simulate(X, y_obs=y, resid=e), reps)
    best_f = min(fwd_ms, key=fwd_ms.get)
    fwd = next(c for c in forward if _name(c) == best_f)
    adj_ms = {}
    for g in adjoint:
        _apply(plan, fwd, g)
        adj_ms[str(g)] = _median_ms(lambda: plan.backproject(e, p, W, num, den), reps)
    best_g = int(min(adj_ms, key=adj_ms.get))
    _apply(plan, fwd, best_g)
    res = {"forward": best_f, "adjoint_granule": best_g, "forward_ms": fwd_ms,
           "adjoint_ms": adj_ms}
    if cache:
        db[key] = res
        _save_cache(cache, db)
    return res
