"""Launch-shape autotuner for the integrate and camera kernels.

Times each candidate launch shape on a sample of the real work (HIP events on the
current stream) and keeps the fastest: the library's default shape (0, 0), threads per
block for malbec_integrate, plus the retire/refill interval (steps_per_chunk) of its
persistent work-queue kernel, and (block, steps_per_chunk) of the persistent camera kernel.
Results are cached per (device, operation, precision, formulation, persistent or not, number
of spacetimes, size bucket) in a JSON file: $MALBEC_TUNE_CACHE, else _build/autotune.json
next to the library.  The binding's integrate() and trace_camera() take a cached shape when
called with block = 0 (and, for persistent launches, steps_per_chunk = 0); without a
cached entry the library's defaults apply: 256 threads per block, lanes that fill the chip
unevenly in turns, a queue only where the lanes are not all in flight at once, refilled
every 64 steps for integrate and every 32 for the camera.  An explicit shape does without
the turns and keeps the queue, so it has to be faster than the default by more than the
timing noise, and it is not taken for lane counts that the default may launch in turns
(a size bucket holds even and uneven ones).  Launch shape never changes results (every
lane's arithmetic is independent of the grid), only speed.
"""
from __future__ import annotations

import json
import os
import threading

import torch

from . import (Camera, _HERE, _spacetimes, integrate, new_lane_arrays, trace_camera)

_lock = threading.Lock()
BLOCKS = (0, 64, 128, 192, 256)  # 0: the library's default
CHUNKS = (0, 8, 32, 128)
_MARGIN = 0.98  # an explicit shape takes at most this share of the default's time
_mem = None  # the cache file's content, loaded once per process
_arch = {}


_default_path = os.path.join(_HERE, "_build", "autotune.json")


def _cache_path():
    return os.environ.get("MALBEC_TUNE_CACHE", _default_path)


def _load():
    global _mem
    path = _cache_path()
    if _mem is None or _mem[0] != path:
        try:
            with open(path) as f:
                _mem = (path, json.load(f))
        except (OSError, ValueError):
            _mem = (path, {})
    return _mem[1]


def _store(cache):
    global _mem
    path = _cache_path()
    os.makedirs(os.path.dirname(path), exist_ok=True)
    tmp = path + ".tmp%d" % os.getpid()
    with open(tmp, "w") as f:
        json.dump(cache, f, indent=1, sort_keys=True)
    os.replace(tmp, path)
    _mem = (path, cache)


def _key(*parts):
    d = torch.cuda.current_device()
    if d not in _arch:
        dev = torch.cuda.get_device_properties(d)
        _arch[d] = getattr(dev, "gcnArchName", dev.name)
    return "|".join([_arch[d]] + [str(p) for p in parts])


def _bucket(n):
    return 1 << max(0, int(n - 1).bit_length())


_thread = threading.local()  # .timing: this thread times candidates, (0, 0) is the default


def _time(fn, reps=2):
    _thread.timing = True
    try:
        fn()  # warm-up
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        best = float("inf")
        for _ in range(reps):
            a.record()
            fn()
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
    finally:
        _thread.timing = False
    return best


def _integrate_key(n, n_st, precision, formulation, persistent):
    return _key("integrate", precision, formulation, "persistent" if persistent else "plain",
                n_st, _bucket(n))


def _shapes(persistent):
    """Candidate (block, steps_per_chunk): the default, then the explicit ones."""
    chunks = CHUNKS[1:] if persistent else (0,)
    return [(0, 0)] + [(b, c) for b in BLOCKS[1:] for c in chunks]


def _best(times):
    best = min(times, key=times.get)
    return best if times[best] < _MARGIN * times[(0, 0)] else (0, 0)


def default_is_better(n, n_steps, precision="f64", persistent=False):
    """Whether the library's default may launch these lanes in turns (FP64, one to nine times the
    256 threads of every CU and up to 0.6 of it more), persistent ones if all are in flight at once."""
    level = 256 * torch.cuda.get_device_properties(torch.cuda.current_device()).multi_processor_count
    w, over = divmod(n, level)
    return precision == "f64" and n_steps >= 100 and 1 <= w <= (2 if persistent else 8) and \
        0 < over <= 0.6 * level


def lookup_integrate(n, n_st, precision="f64", formulation="christoffel", persistent=False):
    """The cached (block, steps_per_chunk) of an integrate launch, or None (no timing)."""
    with _lock:
        cache = _load()
        if not cache or getattr(_thread, "timing", False):  # nothing tuned: no key to build
            return None
        e = cache.get(_integrate_key(n, n_st, precision, formulation, persistent))
    if e and "0,0" not in e.get("ms", {}):  # tuned without the default among the candidates
        return None
    return (e["block"], e["chunk"]) if e else None


def integrate_shape(state, spacetimes, h, precision="f64", formulation="christoffel",
                    persistent=False, st_of_lane=None, probe_steps=200, max_lanes=1 << 18,
                    refresh=False, **kw):
    """Best (block, steps_per_chunk) for malbec_integrate on this batch (cached); (0, 0) is the
    library's default.  For a plain launch the chunk is 0 (all steps in one launch); for the
    persistent kernel it is the retire/refill interval.  Timed on the first max_lanes lanes (with their
    spacetime indices) over probe_steps steps."""
    n = state.shape[-1]
    n_st = len(_spacetimes(spacetimes))
    key = _integrate_key(n, n_st, precision, formulation, persistent)
    with _lock:
        e = _load().get(key)
    if e and "0,0" in e.get("ms", {}) and not refresh:
        return e["block"], e["chunk"]
    m = min(n, max_lanes)
    sample = state[:, :m].contiguous()
    sol = None if st_of_lane is None else st_of_lane[:m].contiguous()
    work = torch.empty_like(sample)
    status, steps = new_lane_arrays(m, device=state.device)
    times = {}
    for blk, ch in _shapes(persistent):
        def run():
            work.copy_(sample)
            status.zero_()
            steps.zero_()
            integrate(work, status, steps, spacetimes, h=h, n_steps=probe_steps,
                      precision=precision, formulation=formulation, persistent=persistent,
                      block=blk, steps_per_chunk=ch, st_of_lane=sol, **kw)
        times[(blk, ch)] = _time(run)
    best = _best(times)
    with _lock:
        cache = dict(_load())
        cache[key] = {"block": best[0], "chunk": best[1],
                      "ms": {"%d,%d" % k: v for k, v in times.items()}}
        _store(cache)
    return best


def integrate_block(state, spacetimes, h, precision="f64", **kw):
    """Best threads per block for a plain integrate launch (integrate_shape's block)."""
    return integrate_shape(state, spacetimes, h, precision=precision, **kw)[0]


def _camera_key(cam: Camera):
    return _key("camera", _bucket(cam.nx * cam.ny), cam.a, cam.max_steps)


def lookup_camera(cam: Camera):
    """The cached (block, steps_per_chunk) of the persistent camera kernel, or None."""
    with _lock:
        e = None if getattr(_thread, "timing", False) else _load().get(_camera_key(cam))
    return tuple(e["shape"]) if e else None


def camera_shape(cam: Camera, sample=1024, refresh=False):
    """Best (block, steps_per_chunk) for the persistent camera kernel (cached), timed on a
    sample x sample image of the same camera (the best of two launches after a warm-up).
    The default 1024 x 1024 sample fills the device several times over, as the full image
    does; on a 256 x 256 one (a single wave per SIMD, 2 ms launches) the choice between
    the shapes, a few per cent apart, followed the timing noise."""
    key = _camera_key(cam)
    with _lock:
        e = _load().get(key)
    if e and not refresh:
        return tuple(e["shape"])
    small = Camera(**{**cam.__dict__, "nx": min(sample, cam.nx), "ny": min(sample, cam.ny),
                      "persistent": 1})
    times = {}
    for blk, ch in _shapes(True):
        c = Camera(**{**small.__dict__, "block": blk, "steps_per_chunk": ch})
        times[(blk, ch)] = _time(lambda: trace_camera(c), reps=2)
    best = _best(times)
    with _lock:
        cache = dict(_load())
        cache[key] = {"shape": list(best), "ms": {"%d,%d" % k: v for k, v in times.items()}}
        _store(cache)
    return best
