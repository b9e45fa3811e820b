"""Tile autotuner for the batched launch (and the per-subdomain kernel).

Times a few steps of the real workload with the automatic launches and for
each candidate tile shape (threads per block, and output rows per tile strip
of the 2-D instances; 1-D tubes always use one-row tiles), and leaves the
fastest in force.  The automatic launches are not among the shapes that can be
set (boxes, two stages or a whole step per launch): where no strip beats them
they stay.  Only speed depends on the shape, never values (every one gives the
same bits), so tuning on the live state is safe.  A JSON cache keyed by the
workload, the device and the built library avoids re-tuning.
"""

from __future__ import annotations

import hashlib
import json
import os
import time
from typing import Dict, Iterable, List, Optional, Sequence, Tuple

import torch

from .sacx import FP32, FP64, LIB_PATH, Batch, Solver

CACHE = os.path.join(os.environ.get("XDG_CACHE_HOME", os.path.expanduser("~/.cache")), "sacx", "autotune.json")


def _load_cache() -> Dict:
    try:
        with open(CACHE) as fh:
            return json.load(fh)
    except (OSError, ValueError):
        return {}


def _save_cache(d: Dict):
    try:
        os.makedirs(os.path.dirname(CACHE), exist_ok=True)
        tmp = CACHE + ".tmp%d" % os.getpid()
        with open(tmp, "w") as fh:
            json.dump(d, fh, indent=1, sort_keys=True)
        os.replace(tmp, CACHE)
    except OSError:
        pass


def _time(fn, reps: int) -> float:
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(reps):
        fn()
    e1.record()
    torch.cuda.synchronize()
    return e0.elapsed_time(e1) / reps


def batch_signature(batch: Batch) -> str:
    g = batch.grids
    return "batch:%d:%s:%s" % (batch.n, "fp64" if g[0].precision == FP64 else "fp32",
                               ",".join("%dx%d" % (g[i].nx, g[i].ny) for i in range(batch.n)))


def _cache_key(batch: Batch) -> str:
    """The workload, the device and the library: shapes timed with another
    build are not taken over."""
    with open(LIB_PATH, "rb") as fh:
        lib = hashlib.sha256(fh.read()).hexdigest()[:16]
    return "%s|%s|%s" % (batch_signature(batch), torch.cuda.get_device_name(batch.device), lib)


def _strip_wins(time_auto, time_strip, rounds: int = 3) -> bool:
    """The two in turn; a strip has to win by more than such short timings scatter."""
    auto, strip = [], []
    for _ in range(rounds):
        auto.append(time_auto())
        strip.append(time_strip())
    return min(strip) < 0.98 * min(auto)


def tune_batch(batch: Batch, threads: Sequence[int] = (128, 256), rows2d: Sequence[int] = (16, 32, 64, 128),
               steps: int = 2, use_cache: bool = True, log=None) -> Tuple[int, int, List[Tuple[int, int, float]]]:
    """Time the automatic launches and every (threads, rows for 2-D instances)
    of a batch and leave the fastest in force (batch.tiles: None where the
    automatic launches stay).  Returns the fastest shape that can be set and
    the trials, the automatic launches among them as (0, 0, ms).  Advances the
    batch by (1 + steps) x (number of candidates + 1) steps while measuring, and
    six times 1 + steps more where a strip comes in front."""
    key = _cache_key(batch) if use_cache else ""
    cache = _load_cache() if use_cache else {}

    def apply(t, r):
        if t:
            batch.set_tiles(t, [r] * batch.n)
        else:
            batch.set_tiles_auto()

    if key in cache:
        t, r = cache[key]["threads"], cache[key]["rows2d"]
        if cache[key]["automatic"]:
            apply(0, 0)
        else:
            apply(t, r)
        return t, r, []

    def timed(t, r):
        apply(t, r)
        batch.advance(1, sync=True)                     # table build + warm-up
        return _time(lambda: batch.advance(steps, sync=False), 1) / steps

    trials = []
    for t, r in [(0, 0)] + [(t, r) for t in threads for r in rows2d]:
        ms = timed(t, r)
        trials.append((t, r, ms))
        if log:
            log(f"[autotune] threads={t} rows={r}: {ms:.3f} ms/step" if t else f"[autotune] automatic: {ms:.3f} ms/step")
    t, r, ms = min(trials[1:], key=lambda x: x[2])
    automatic = not (ms < trials[0][2] and _strip_wins(lambda: timed(0, 0), lambda: timed(t, r)))
    apply(*((0, 0) if automatic else (t, r)))
    if use_cache:
        cache[key] = {"threads": t, "rows2d": r, "automatic": automatic, "trials": trials}
        _save_cache(cache)
    return t, r, trials


def tune_solver(s: Solver, threads: Sequence[int] = (64, 128, 256), rows: Sequence[int] = (32, 64, 128, 256),
                log=None) -> Tuple[int, int]:
    """Time the automatic launches and every launch shape of one subdomain, and
    leave the fastest in force.  Returns the fastest shape that can be set.
    Steps are timed two to a call: the automatic launches of some grids take
    steps in pairs."""

    def timed(t, r):
        if t:
            s.set_launch(t, r)
        else:
            s.set_launch_auto()
        s.advance(2)
        return _time(lambda: s.advance(2, sync=False), 2) / 2

    auto = timed(0, 0)
    if log:
        log(f"[autotune] automatic: {auto:.3f} ms/step")
    best = None
    for t in threads:
        for r in rows:
            try:
                s.set_launch(t, r)
            except Exception:
                continue
            ms = timed(t, r)
            if log:
                log(f"[autotune] threads={t} rows={r}: {ms:.3f} ms/step")
            if best is None or ms < best[2]:
                best = (t, r, ms)
    if best[2] < auto and _strip_wins(lambda: timed(0, 0), lambda: timed(best[0], best[1])):
        s.set_launch(best[0], best[1])
    else:
        s.set_launch_auto()
    return best[0], best[1]
