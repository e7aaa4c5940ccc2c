"""Autotuner for the library's launch parameters (hawkes_set_tuning).

For a problem shape it times each candidate setting on the caller's own
inputs (a few calls each, device time from HIP events on the current
stream), checks that every candidate reproduces the default setting's
log-likelihood and every gradient block to rounding, keeps the fastest (the library's own rule unless a
candidate is at least 1% faster), applies it with
``set_tuning`` and stores it in a JSON cache keyed by the device and a shape
class, so that later processes skip the timing.

Knobs (see include/hawkes.h):
  dense_cols, dense_ranges   the shared-decay large-M engine (M > 64, or several
                             decay kernels): events per block and event ranges
                             of the dense dL/dalpha
  item_log2                  the small-M engine (M <= 8, single or batched):
                             events per lane item

The per-target engine and the one for 9 to 64 nodes and one shared decay have no
knobs.  The cache file is
$HAWKES_TUNE_CACHE, else ~/.cache/paper_2604_01342_amd/tuning.json.
"""
from __future__ import annotations

import json
import math
import os
from typing import Callable, Iterable

import torch

from . import Batch, get_tuning, loglik_grad, loglik_grad_batched, set_tuning

# candidates must agree with the default setting to rounding, per output
# block (normwise relative): the log-likelihood, dL/dmu and dL/dbeta are
# float64 sums whose order the layouts change; dL/dalpha of the dense
# kernels also uses float32 decay factors against anchors that the layout
# places (a few float32 ulp each), so it agrees to about 1e-8
TOL = {"loglik": 1e-9, "g_mu": 1e-9, "g_alpha": 2e-7, "g_beta": 1e-9}
MARGIN = 0.01  # a candidate replaces the library's rule only when at least 1% faster
               # (equal layouts, or timing noise, keep the rule)


def cache_path() -> str:
    return os.environ.get("HAWKES_TUNE_CACHE") or os.path.join(
        os.path.expanduser("~"), ".cache", "paper_2604_01342_amd", "tuning.json")


def _device_key(dev) -> str:
    p = torch.cuda.get_device_properties(dev)
    return f"{p.name}|{getattr(p, 'gcnArchName', '')}|{p.multi_processor_count}"


def _bucket(x: int) -> int:
    return int(math.floor(math.log2(max(1, x))))


def _narrow(M: int, per_target: bool, K: int) -> bool:
    """Shapes that one kernel takes (9 to 64 nodes, one shared decay)."""
    return not per_target and K == 1 and 8 < M <= 64


def shape_class_single(n: int, M: int, per_target: bool, chunk_log2: int, K: int = 1) -> str:
    """Shapes that share a setting: M and n by powers of two, the decay mode,
    the chunk size.  The shapes of one kernel have classes of their own; so have
    those of the dense kernels' event blocks ("blk2"): settings stored for
    earlier forms of these kernels are not taken up."""
    kind = "|narrow" if _narrow(M, per_target, K) else "|blk2" if M > 8 and not per_target else ""
    return f"single|M{_bucket(M)}|n{_bucket(n)}|pt{int(per_target)}|ch{chunk_log2 or 20}{kind}"


def shape_class_batched(S: int, n_total: int, max_m: int) -> str:
    return f"batched|S{_bucket(S)}|n{_bucket(n_total)}|M{_bucket(max_m)}"


def candidates_single(n: int, M: int, per_target: bool, chunk_log2: int, K: int = 1) -> list[dict]:
    if per_target or _narrow(M, per_target, K):
        return [{}]
    if M <= 8:
        return [{"item_log2": k} for k in range(4, 11)]
    return [{"dense_cols": c, "dense_ranges": r} for c in (64, 128, 256) for r in (2, 4, 8, 16, 32)]


def candidates_batched(n_total: int) -> list[dict]:
    return [{"item_log2": k} for k in range(5, 12)]


def _load() -> dict:
    try:
        with open(cache_path()) as f:
            return json.load(f)
    except (OSError, ValueError):
        return {}


def _store(cache: dict) -> bool:
    """Write the cache; False (and no cache) where the path is not writable."""
    path = cache_path()
    try:
        os.makedirs(os.path.dirname(path), exist_ok=True)
        tmp = f"{path}.tmp{os.getpid()}"
        with open(tmp, "w") as f:
            json.dump(cache, f, indent=1, sort_keys=True)
        os.replace(tmp, path)
        return True
    except OSError:
        return False


def _time_ms(fn: Callable[[], object], reps: int) -> float:
    fn()   # warm (and size the workspace)
    torch.cuda.synchronize()
    best = float("inf")
    for _ in range(reps):
        a = torch.cuda.Event(enable_timing=True)
        b = torch.cuda.Event(enable_timing=True)
        a.record()
        fn()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


def _blocks_differ(got, ref) -> str | None:
    """The first output block whose normwise relative difference from the
    default setting's exceeds its TOL (or is not finite), described, else None."""
    for name, a, b in zip(("loglik", "g_mu", "g_alpha", "g_beta"), got, ref):
        a = a.double().reshape(-1)
        b = b.double().reshape(-1)
        if not bool(torch.isfinite(a).all()):
            return f"{name} (not finite)"
        nb = float(torch.linalg.vector_norm(b))
        d = float(torch.linalg.vector_norm(a - b)) / max(nb, 1e-300)
        if d > TOL[name]:
            return f"{name} by {d:.3e} relative (limit {TOL[name]:.0e})"
    return None


def _search(key: str, cands: Iterable[dict], run: Callable[[], tuple], reps: int, use_cache: bool,
            log: Callable[[str], None] | None) -> dict:
    dev = torch.cuda.current_device()
    dkey = _device_key(dev)
    cache = _load() if use_cache else {}
    hit = cache.get(dkey, {}).get(key)
    if hit is not None:
        set_tuning(**hit["tuning"])
        return hit
    set_tuning()
    ref = [x.clone() for x in run()]
    results = []
    for c in cands:
        set_tuning(**c)
        bad = _blocks_differ(run(), ref)
        if bad is not None:
            set_tuning()
            raise RuntimeError(f"tuning {c} changed {bad}")
        ms = _time_ms(run, reps)
        results.append((ms, c))
        if log:
            log(f"tune {key}: {c} {ms:.3f} ms")
    set_tuning()
    base_ms = _time_ms(run, reps)
    ms, best = min(results, key=lambda r: r[0])
    if ms > base_ms * (1.0 - MARGIN):
        ms, best = base_ms, {}
    out = {"tuning": {"dense_cols": best.get("dense_cols", 0), "dense_ranges": best.get("dense_ranges", 0),
                      "item_log2": best.get("item_log2", 0), "dense_rows": best.get("dense_rows", 0)},
           "ms": ms, "default_ms": base_ms}
    set_tuning(**out["tuning"])
    if use_cache:
        cache.setdefault(dkey, {})[key] = out
        _store(cache)
    return out


def tune_single(t, m, mu, alpha, beta, T, chunk_log2: int = 0, reps: int = 3, use_cache: bool = True,
                log: Callable[[str], None] | None = None) -> dict:
    """Choose and apply the setting for loglik_grad on this sequence; returns
    {"tuning": ..., "ms": best time per call, "default_ms": the library's own
    rule}.  The inputs must be on the GPU."""
    M = int(mu.numel())
    per_target = int(beta.numel()) == M and M > 1
    n = int(t.numel())
    K = int(alpha.numel()) // (M * M)
    key = shape_class_single(n, M, per_target, chunk_log2, K)

    def run() -> tuple:
        L, gmu, ga, gb = loglik_grad(t, m, mu, alpha, beta, T, chunk_log2)
        return L.reshape(1), gmu, ga, gb

    return _search(key, candidates_single(n, M, per_target, chunk_log2, K), run, reps, use_cache, log)


def tune_batched(b: Batch, reps: int = 3, use_cache: bool = True,
                 log: Callable[[str], None] | None = None) -> dict:
    """Choose and apply the item length for loglik_grad_batched on this batch."""
    n_total = int(b.t.numel())
    key = shape_class_batched(b.S, n_total, b.max_m)

    def run() -> tuple:
        return loglik_grad_batched(b)

    return _search(key, candidates_batched(n_total), run, reps, use_cache, log)


def current() -> dict:
    return get_tuning()
