"""Autotuned plans, cached on disk per device architecture.

`tune(limbs, kind, exp_bits, count)` runs the library's autotuner
(rsa_autotune: every compiled kernel instance of the width class at every
window that fits, and the RNS kernels where they serve the call, timed on
synthetic operands of the given batch size: plain calls for kinds 0 and 1,
rsa_ops_batch on a synthetic keyset for kinds 2 to 4) and records the winner,
plan and path, in a JSON cache; `apply_cached()` re-installs cached entries so
later processes skip the search.  An entry without a path, of a search among
the positional kernels alone, leaves RNS the calls it serves.  Entries are
keyed by the GPU architecture, the operand width in words, the kind, the
exponent length and the batch size rounded up to a power of two.

`tune_batch(run, slots)` tunes the plans of a whole rsa_ops_batch call
jointly: the buckets of a mixed batch run side by side and compete for the
CUs (registers, LDS, issue slots), so the plan that is fastest for a bucket
alone (often the one with the shortest chain) need not be the fastest in the
mix.  It installs each candidate plan of one (width, kind) slot at a time
and times the real call, keeping the fastest (coordinate descent).
"""
from __future__ import annotations

import json
import os
from typing import Dict, Optional

import torch

from . import rsagpu

_DEFAULT = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), ".tunecache",
                        "plans.json")


def cache_path() -> str:
    return os.environ.get("RSAGPU_TUNE_FILE", _DEFAULT)


def _arch() -> str:
    return torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]


CRT_KINDS = (1, 3, 4)


def plan_width(limbs: int, kind: int) -> int:
    """Width whose class a plan of `kind` is stored under (CRT: one half)."""
    return limbs // 2 if kind in CRT_KINDS else limbs


def _key(limbs: int, kind: int, exp_bits: int, count: int) -> str:
    bucket = 1 << max(0, (count - 1).bit_length())
    return "%s/w%d/k%d/e%d/n%d" % (_arch(), limbs, kind, exp_bits, bucket)


def load() -> Dict[str, dict]:
    try:
        with open(cache_path()) as f:
            return json.load(f)
    except (OSError, ValueError):
        return {}


def save(cache: Dict[str, dict]) -> None:
    path = cache_path()
    os.makedirs(os.path.dirname(path), exist_ok=True)
    tmp = path + ".tmp%d" % os.getpid()
    with open(tmp, "w") as f:
        json.dump(cache, f, indent=1, sort_keys=True)
    os.replace(tmp, path)


def _install(width: int, kind: int, entry: dict) -> None:
    rsagpu.set_plan(width, kind, entry["radix_bits"], entry["lanes_per_op"], entry["window_bits"])
    rsagpu.set_path(width, kind, entry.get("path", rsagpu.PATH_AUTO))


def tune(limbs: int, kind: int, exp_bits: int, count: int, use_cache: bool = True) -> rsagpu.Plan:
    """Best plan for (limbs, kind, exp_bits, count), installed in the library."""
    cache = load()
    key = _key(limbs, kind, exp_bits, count)
    width = plan_width(limbs, kind)
    if use_cache and key in cache:
        _install(width, kind, cache[key])
        return rsagpu.get_plan(width, kind)
    plan = rsagpu.autotune(limbs, kind, exp_bits, count)
    cache[key] = {"radix_bits": plan.radix_bits, "lanes_per_op": plan.lanes_per_op,
                  "window_bits": plan.window_bits, "padded_limbs": plan.padded_limbs,
                  "path": rsagpu.get_path(width, kind)}
    save(cache)
    return plan


def apply_cached(arch: Optional[str] = None) -> int:
    """Installs every cached plan of this architecture; returns how many."""
    arch = arch or _arch()
    n = 0
    for key, e in load().items():
        parts = key.split("/")
        if parts[0] != arch:
            continue
        limbs, kind = int(parts[1][1:]), int(parts[2][1:])
        width = plan_width(limbs, kind)
        _install(width, kind, e)
        n += 1
    return n


def candidate_plans(width: int, kind: int):
    """(radix_bits, lanes_per_op, window_bits) the library accepts for the
    width class of `width` and plan `kind` (the current plan is restored;
    none where the class has no plan of that kind)."""
    try:
        cur, path = rsagpu.get_plan(width, kind), rsagpu.get_path(width, kind)
    except rsagpu.RSAError:
        return []
    out = []
    for radix in (32, 29):
        for lanes in (1, 2, 4, 8, 16):
            for w in range(2, 7):
                try:
                    rsagpu.set_plan(width, kind, radix, lanes, w)
                except rsagpu.RSAError:
                    continue
                out.append((radix, lanes, w))
    rsagpu.set_plan(width, kind, cur.radix_bits, cur.lanes_per_op, cur.window_bits)
    rsagpu.set_path(width, kind, path)
    return out


def tune_batch(run, slots, reps: int = 3, passes: int = 1, tolerance: float = 0.005, knobs=(),
               timer=None, confirm: int = 5):
    """Coordinate descent over the plans of `slots` [(width, kind), ...] for
    the batch that run() enqueues on torch's current stream: each candidate
    (a plan, which runs positionally; the slot's starting plan and path; and,
    where that is RNS, the starting plan positionally, given as (radix, lanes,
    window, "positional")) is installed and the batch timed (one warm-up, then `reps` runs between
    HIP events); a candidate replaces the slot's plan when it is faster by
    more than `tolerance` in two timings in a row (one lucky timing does not
    move the descent).  `knobs` [(name, values, apply)] are further settings
    tuned the same way after the plans (apply(value) installs one; values[0]
    is the current one).  At the end the starting settings and the chosen
    ones are timed `confirm` times each, alternately, and the chosen ones are
    kept only if their median is faster by more than `tolerance`; otherwise
    the starting settings are restored.  `timer`, if given, replaces the HIP
    event timing (a callable returning ms per call).  Returns ({(width,
    kind): (radix, lanes, window), name: value, ...}, ms per call with the
    settings in place)."""
    if timer is None:
        stream = torch.cuda.current_stream()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)

        def timer() -> float:
            run()
            e0.record(stream)
            for _ in range(reps):
                run()
            e1.record(stream)
            e1.synchronize()
            return e0.elapsed_time(e1) / reps

    def plan_of(width, kind):
        p = rsagpu.get_plan(width, kind)
        return (p.radix_bits, p.lanes_per_op, p.window_bits)

    def put(slot, value):
        rsagpu.set_plan(*slot, *value[:3])
        if value == start[slot]:
            rsagpu.set_path(*slot, path[slot])

    def install(cfg):
        for key, value in cfg.items():
            if isinstance(key, tuple):
                put(key, value)
        for name, _, apply in knobs:
            apply(cfg[name])

    def candidates(slot):
        yield from candidate_plans(*slot)
        if path[slot] == rsagpu.PATH_AUTO and slot[1] in CRT_KINDS[1:] and \
                rsagpu.get_path(*slot, 1) == rsagpu.PATH_RNS:
            yield start[slot] + ("positional",)

    start = {(w, k): plan_of(w, k) for w, k in slots}
    path = {(w, k): rsagpu.get_path(w, k) for w, k in slots}
    for name, values, _ in knobs:
        start[name] = values[0]

    def better(ms, best):
        return ms < best * (1.0 - tolerance)

    best = timer()
    chosen = dict(start)
    for _ in range(passes):
        for width, kind in slots:
            cur = chosen[(width, kind)]
            for cand in list(candidates((width, kind))):
                if cand == cur:
                    continue
                put((width, kind), cand)
                ms = timer()
                if better(ms, best):
                    ms2 = timer()
                    if better(ms2, best):
                        best, cur = max(ms, ms2), cand
            put((width, kind), cur)
            chosen[(width, kind)] = cur
        for name, values, apply in knobs:
            cur = chosen[name]
            for v in values:
                if v == cur:
                    continue
                apply(v)
                ms = timer()
                if better(ms, best):
                    ms2 = timer()
                    if better(ms2, best):
                        best, cur = max(ms, ms2), v
            apply(cur)
            chosen[name] = cur
    if chosen == start:
        return chosen, best
    a, b = [], []
    for _ in range(confirm):
        install(start)
        a.append(timer())
        install(chosen)
        b.append(timer())
    a.sort()
    b.sort()
    if better(b[len(b) // 2], a[len(a) // 2]):
        return chosen, b[len(b) // 2]
    install(start)
    return dict(start), a[len(a) // 2]
