"""Autotuner of the sweep launch: tile shape and plane chunks per level.

It times whole runs, as they will be launched: one compiled tile shape (rows
per wave x waves per workgroup) on every level after another; for a grid config
of two levels also the mix of shapes that each level's own launch is fastest
with (its launches timed one by one by the library's HIP events); then, level by
level, each plane-chunk count.  The fastest of each is kept.  A persistent
config's shapes are ranked by its sweep launch, the only one that they change.
The choice is remembered in a JSON cache keyed by the device, the level shapes,
the source count, the staging precision and the launch kind.  Deterministic: a
cached choice is reused as is."""
from __future__ import annotations

import json
import os

import torch

from .sweep import PlaneSweep

CANDIDATES = [(4, 4), (8, 4), (4, 8), (2, 8), (16, 4), (8, 2)]
CHUNK_CANDIDATES = [0, 1, 2, 3, 4, 6, 8]  # 0: the library's automatic count
DEFAULT_CACHE = os.path.join(os.path.expanduser("~"), ".cache", "psweep_tiles.json")


def _key(sweep: PlaneSweep, frames) -> str:
    props = torch.cuda.get_device_properties(sweep.device)
    lv = ";".join(f"{l.n_fronto}+{l.n_ground}w{l.window}d{l.downsample}c{tuple(l.crop)}" for l in sweep.settings.levels)
    sizes = ",".join(f"{f['ref'].shape[1]}x{f['ref'].shape[0]}" for f in frames)
    return (f"{props.gcnArchName}|{lv}|S{len(frames[0]['srcs'])}|st{sweep.cfg.storage}|"
            f"launch{sweep.cfg.launch}|{sizes}|runs")   # ranked by whole runs: older choices are not


def _time(sweep, frames, outputs, reps):
    sweep.set_timing(True)
    best = float("inf")
    try:
        for _ in range(reps):
            sweep.run(frames, outputs)
            torch.cuda.synchronize()
            ms, n = sweep.sweep_kernel_ms()
            best = min(best, ms * n)
    finally:   # a shape that is not compiled ends here too
        sweep.set_timing(False)
    return best


def _run_ms(sweep, frames, outputs, reps):
    """Fastest whole run (every kernel of psweep_run), HIP events on the
    launch stream.  A run goes before the one that is timed, so that the host's
    part of that one lies beside the GPU's work."""
    best = float("inf")
    for _ in range(reps):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        sweep.run(frames, outputs)
        e0.record()
        sweep.run(frames, outputs)
        e1.record()
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1))
    return best


def _level_ms(sweep, frames, outputs):
    """Durations of each sweep launch of a timed run: a grid config then
    launches its (frame, level) jobs one by one, in that order."""
    sweep.set_timing(True)
    try:
        sweep.run(frames, outputs)
        torch.cuda.synchronize()
    finally:
        sweep.set_timing(False)
    from . import psweep as P
    return P.psweep_sweep_kernel_times(sweep.ctx)


def _set_tiles(sweep, tiles):
    for l, (r, w) in enumerate(tiles):
        sweep.set_tile(l, r, w)


def _apply(sweep, choice):
    _set_tiles(sweep, choice["tiles"])
    for l, c in enumerate(choice.get("chunks", [0] * len(choice["tiles"]))):
        sweep.set_chunks(l, c)


def tune(sweep: PlaneSweep, frames, outputs, reps: int = 5, cache_path: str | None = DEFAULT_CACHE,
         candidates=CANDIDATES, chunk_candidates=CHUNK_CANDIDATES) -> dict:
    """Pick a tile shape per level (one shape for all levels with the
    persistent launch), then a plane-chunk count per level.  Returns {"key":
    ..., "tiles": [[rows, waves], ...], "chunks": [...], "ms": ..., "run_ms":
    ...} and applies it to `sweep`.  "ms": what the tiles were ranked by."""
    key = _key(sweep, frames)
    cache = {}
    if cache_path and os.path.exists(cache_path):
        try:
            with open(cache_path) as f:
                cache = json.load(f)
        except (OSError, ValueError):
            cache = {}
    nl = len(sweep.settings.levels)
    if key in cache:
        choice = cache[key]
        _apply(sweep, choice)
        return choice
    persistent = sweep.cfg.launch == 1
    measure = _time if persistent else _run_ms
    results = {}
    for cand in candidates:
        try:
            _set_tiles(sweep, [cand] * nl)
            results[cand] = measure(sweep, frames, outputs, reps)
        except Exception:   # shape not compiled for this window / source count
            results[cand] = float("inf")
    best = min(results, key=results.get)
    tiles, ms = [list(best)] * nl, results[best]
    if nl > 1 and not persistent:
        # Each level's own fastest shape.  Where they differ the run is a launch
        # per job, which can be slower than one launch of one shape: the mix is
        # kept only if its whole run is faster (16 frames of two levels, four
        # sources, FP32: the mix 14.9 ms, one shape 12.8).
        per_level = {}
        for cand, t in results.items():
            if t < float("inf"):
                _set_tiles(sweep, [cand] * nl)
                per_level[cand] = _level_ms(sweep, frames, outputs)
        mix = [list(min(per_level, key=lambda c: per_level[c][l] if l < len(per_level[c]) else float("inf")))
               for l in range(nl)] if per_level else tiles
        if mix != [mix[0]] * nl:
            _set_tiles(sweep, mix)
            t = _run_ms(sweep, frames, outputs, reps)
            results["mix"] = t
            if t < ms:
                tiles, ms = mix, t
    _set_tiles(sweep, tiles)
    # plane chunks, level by level, on whole-run time (the combine of chunks
    # is a kernel of its own)
    chunks, chunk_ms = [], {}
    for l in range(nl):
        best_c, best_t = 0, float("inf")
        for c in chunk_candidates:
            sweep.set_chunks(l, c)
            t = _run_ms(sweep, frames, outputs, reps)
            chunk_ms[f"level{l}:{c}"] = t
            if t < best_t:
                best_c, best_t = c, t
        sweep.set_chunks(l, best_c)
        chunks.append(best_c)
    choice = {"key": key, "tiles": tiles, "chunks": chunks, "ms": ms, "run_ms": min(chunk_ms.values()),
              "candidates": {c if c == "mix" else f"{c[0]}x{c[1]}": v for c, v in results.items()},
              "chunk_candidates": chunk_ms}
    if cache_path:
        cache[key] = choice
        os.makedirs(os.path.dirname(cache_path), exist_ok=True)
        tmp = cache_path + ".tmp"
        with open(tmp, "w") as f:
            json.dump(cache, f, indent=1, sort_keys=True)
        os.replace(tmp, cache_path)
    return choice
