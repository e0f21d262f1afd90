"""Autotuner for the batched sampler's launch shape.

Times whole batched steps on the device on a scratch batch holding the
caller's workload shapes, for the knobs that change only speed (every
candidate gives the same bits):

  - ``k_bprop`` / unit_pairs: coordinate pairs per proposal work unit.  The
    proposal has no units any more, so the choice is fixed and one timing of the
    step stands for every candidate;
  - ``k_bquad`` / waves, per dimension bucket: the occupancy the target
    kernel of samplers with d in (8 q, 8 q + 8] aims at (1 up to that
    bucket's highest, where the bucket joins the others in one launch), tuned
    one bucket at a time with the others at their current choice, the
    candidates timed in turn.

Results are kept in a JSON cache keyed by kernel, knob, bucket, device
architecture (gcnArchName, e.g. gfx950), a digest of the workload's (N, d)
shapes and the version of what a choice means (``RULE``), so a later run on the
same device and workload reuses them without timing.  The cache file is ``$SMC_TUNE_CACHE`` or
``~/.cache/paper_1905_10252_amd/tune.json``.
"""
from __future__ import annotations

import hashlib
import json
import os
import statistics

import torch

from . import smc

GROUP_CANDIDATES = (2, 4, 5, 6, 8)
GROUP_DEFAULT = 8  # what a batch starts with
BUCKETS = 8
ROUNDS = 4  # timings of a candidate
# What a cached choice means, raised with the kernels or the rule that picked it.
# 2: an aim below the bucket's highest takes the bucket out of the common launch (the
# entries before, without a version, chose among launches of the bucket's own).
RULE = 2


def _max_waves(bucket: int) -> int:
    d = 8 * (bucket + 1)
    return 4 if d <= 40 else 3


def cache_path() -> str:
    return os.environ.get("SMC_TUNE_CACHE") or os.path.join(
        os.path.expanduser("~"), ".cache", "paper_1905_10252_amd", "tune.json")


def _load(path: str) -> dict:
    try:
        with open(path) as f:
            return json.load(f)
    except (OSError, ValueError):
        return {}


def _store(path: str, data: dict) -> None:
    try:
        os.makedirs(os.path.dirname(path), exist_ok=True)
        tmp = path + ".tmp%d" % os.getpid()
        with open(tmp, "w") as f:
            json.dump(data, f, indent=1, sort_keys=True)
        os.replace(tmp, path)
    except OSError:
        pass  # an unwritable cache only costs a retune next time


def arch(dev) -> str:
    return torch.cuda.get_device_properties(dev).gcnArchName.split(":")[0]


def workload_digest(specs) -> str:
    shapes = sorted((int(sp["n"]), int(sp["d"])) for sp in specs)
    return hashlib.sha1(repr(shapes).encode()).hexdigest()[:16]


def key(kernel: str, knob: str, bucket, arch_name: str, digest: str) -> str:
    return "%s|%s|%s|%s|%s|rule%d" % (kernel, knob, "all" if bucket is None else bucket, arch_name,
                                      digest, RULE)


def _scratch_batch(specs, dev):
    b = smc.Batch(len(specs), graph=False, device=dev)
    for k, sp in enumerate(specs):
        b.attach(k, sp["n"], sp["d"], sp["mean"], sp["chol"], seed=sp["seed"],
                 sampler_id=sp["sampler_id"], rw_sd=sp["rw_sd"], init_sd=sp.get("init_sd", 3.0))
    return b


def _time_steps(b, steps: int) -> float:
    b.step(info=False, est=False)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(steps):
        b.step(info=False, est=False)
    e1.record()
    torch.cuda.synchronize()
    return e0.elapsed_time(e1) / steps


def _in_turn(candidates, timing) -> dict:
    """ROUNDS timings of every candidate, all of them in each round, every other round
    backwards: the clock's drift over a run (9 % over five timings of one and the
    same step) then falls on all alike."""
    candidates = list(candidates)
    times = {c: [] for c in candidates}
    for r in range(ROUNDS):
        for c in candidates if r % 2 == 0 else reversed(candidates):
            times[c].append(timing(c))
    return times


def _faster_than(top, times: dict):
    """The fastest candidate that beats `top` by 2 % in the mean of every pair of rounds,
    forwards and backwards, else `top`.  A lower aim takes its bucket out of the
    common launch: only for a gain that no drift or stray timing makes up."""
    def pairs(c):
        return [times[c][r] + times[c][r + 1] for r in range(0, ROUNDS, 2)]
    ref = pairs(top)
    sure = [c for c in times if all(a < 0.98 * b for a, b in zip(pairs(c), ref))]
    return min(sure, key=lambda c: statistics.median(times[c])) if sure else top


def tune_group(specs, *, device=None, steps: int = 3, candidates=GROUP_CANDIDATES,
               use_cache: bool = True) -> dict:
    """``specs``: sampler descriptions (dicts with n, d, mean, chol, seed,
    sampler_id, rw_sd, init_sd).  Returns {"best": pairs, "ms": {pairs: ms},
    "cached": bool}.  The library ignores the pairs: "best" is GROUP_DEFAULT where
    that is a candidate, and every candidate has the same "ms"."""
    dev = torch.device(device or "cuda")
    path, k = cache_path(), key("k_bprop", "unit_pairs", None, arch(dev), workload_digest(specs))
    data = _load(path) if use_cache else {}
    if k in data:
        return {"best": data[k]["best"], "ms": data[k]["ms"], "cached": True}
    candidates = list(candidates)
    times = dict.fromkeys(candidates, _time_steps(_scratch_batch(specs, dev), steps))
    best = GROUP_DEFAULT if GROUP_DEFAULT in candidates else candidates[0]
    if use_cache:
        data = _load(path)
        data[k] = {"best": best, "ms": {str(g): t for g, t in times.items()}}
        _store(path, data)
    return {"best": best, "ms": times, "cached": False}


def tune_buckets(specs, *, device=None, steps: int = 4, pairs: int | None = None,
                 use_cache: bool = True) -> dict:
    """Occupancy aim of the target kernel per dimension bucket present in the
    workload (one bucket at a time, whole-step timings).  Returns
    {"best": {bucket: waves}, "ms": {bucket: {waves: ms}}, "cached": [...]}."""
    dev = torch.device(device or "cuda")
    a, dg = arch(dev), workload_digest(specs)
    path = cache_path()
    data = _load(path) if use_cache else {}
    present = sorted({(int(sp["d"]) - 1) // 8 for sp in specs})
    best, ms, cached = {}, {}, []
    todo = []
    for q in present:
        k = key("k_bquad", "waves", q, a, dg)
        if k in data:
            best[q] = data[k]["best"]
            ms[q] = data[k]["ms"]
            cached.append(q)
        else:
            best[q] = _max_waves(q)
            todo.append(q)
    if todo:
        b = _scratch_batch(specs, dev)
        if pairs is not None:
            b.set_group(pairs)
        for q in present:
            b.set_bucket_waves(q, best[q])
        for q in todo:
            times = _in_turn(range(1, _max_waves(q) + 1),
                             lambda w: (b.set_bucket_waves(q, w), _time_steps(b, steps))[1])
            best[q] = _faster_than(_max_waves(q), times)
            b.set_bucket_waves(q, best[q])
            ms[q] = {w: statistics.median(t) for w, t in times.items()}
        del b
        if use_cache:
            data = _load(path)
            for q in todo:
                data[key("k_bquad", "waves", q, a, dg)] = {
                    "best": best[q], "ms": {str(w): t for w, t in ms[q].items()}}
            _store(path, data)
    return {"best": best, "ms": ms, "cached": cached}


def apply(batch, tuned_group: dict | None = None, tuned_buckets: dict | None = None) -> None:
    """Sets a batch's knobs to tuned choices."""
    if tuned_group is not None:
        batch.set_group(tuned_group["best"])
    if tuned_buckets is not None:
        for q, w in tuned_buckets["best"].items():
            batch.set_bucket_waves(int(q), int(w))
