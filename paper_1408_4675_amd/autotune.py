"""FFT schedule autotuner.

For each axis of a grid it times candidate radix schedules (and, for the
column passes, column-tile widths; for the x rows, rows per block) with the
library's per-kernel HIP-event profiling, keeps the fastest, and caches the
choice as JSON keyed by device architecture, axis kind and transform length.
`Simulation` applies cached choices automatically: as hints, which serve the
passes on the radix-pass engines and leave those on staged transforms (with
schedules of their own) where they are, or, where the step was measured faster
with the schedule than with the library's defaults, by force; without a cache
the defaults are used.  This plays the role that FFT planning by measurement plays in the paper's cluster code (Section 3.4), but the search
space is this library's own: radix factorisations 2/3/4/5/8/16(/32) and tile
shapes of the LDS-staged passes.
"""
from __future__ import annotations

import itertools
import json
import os
from typing import Dict, List, Optional, Sequence, Set, Tuple

CACHE_ENV = "KW_TUNE_CACHE"
DEFAULT_CACHE = os.path.join(os.path.expanduser("~"), ".cache", "kw_tune.json")

# kernel classes whose time depends on each axis' schedule
AXIS_CLASSES = {0: ("xvel", "xden", "xeos"),
                1: ("ypass_fwd", "ypass_inv"),
                2: ("zfused_grad", "zfused_div", "zfused_abs")}


def cache_path() -> str:
    return os.environ.get(CACHE_ENV, DEFAULT_CACHE)


def _arch() -> str:
    try:
        import torch
        return torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    except Exception:
        return "unknown"


def load_cache() -> Dict:
    p = cache_path()
    if os.path.exists(p):
        try:
            with open(p) as fh:
                return json.load(fh)
        except (OSError, ValueError):
            return {}
    return {}


def save_cache(d: Dict):
    p = cache_path()
    os.makedirs(os.path.dirname(p), exist_ok=True)
    tmp = p + ".tmp"
    with open(tmp, "w") as fh:
        json.dump(d, fh, indent=1, sort_keys=True)
    os.replace(tmp, p)


def key(axis: int, n: int, arch: Optional[str] = None) -> str:
    return "%s|%s|%d" % (arch or _arch(), "xyz"[axis], n)


SHIPPED_DIR = os.path.join(os.path.dirname(os.path.abspath(__file__)), "tuning")


def shipped_table(arch: Optional[str] = None) -> Dict:
    """Choices measured for this package on `arch` and shipped with it."""
    p = os.path.join(SHIPPED_DIR, "%s.json" % (arch or _arch()))
    if os.path.exists(p):
        with open(p) as fh:
            return json.load(fh)
    return {}


def lengths(grid) -> Tuple[int, int, int]:
    """Transform length per axis: nx/2 for the packed x rows, ny, nz."""
    return (grid.nx // 2, grid.ny, grid.nz)


def _factorisations(n: int, radices: Sequence[int], max_passes: int = 4) -> List[List[int]]:
    out = []

    def rec(m, cur):
        if m == 1:
            out.append(list(cur))
            return
        if len(cur) >= max_passes:
            return
        for r in radices:
            if m % r == 0 and (not cur or r <= cur[-1]):
                cur.append(r)
                rec(m // r, cur)
                cur.pop()
    rec(n, [])
    return out


def candidates(axis: int, n: int) -> List[Tuple[List[int], int]]:
    """(radix schedule, tile) pairs worth timing for one axis."""
    pow2 = n & (n - 1) == 0
    if pow2:
        scheds = _factorisations(n, (16, 8, 4, 2), 4)
        # keep the shortest schedules (at most one pass more than the minimum)
        mn = min(len(s) for s in scheds)
        scheds = [s for s in scheds if len(s) <= mn + 1]
        if n >= 32:
            # the 32-wide fixed engine: radix-32 passes only
            scheds += _factorisations(n, (32,), 3)
        # the four-wide fixed engine (radices up to 4: more passes, fewer
        # registers per thread)
        four = _factorisations(n, (4, 2), 8)
        if four:
            mn4 = min(len(s) for s in four)
            scheds += [s for s in four if len(s) == mn4 and s not in scheds][:1]
    else:
        scheds = _factorisations(n, (16, 15, 12, 10, 8, 6, 5, 4, 3, 2), 3)
        mn = min(len(s) for s in scheds)
        scheds = [s for s in scheds if len(s) == mn][:6]
        # the mixed-radix fixed engine (12 or 20 elements per thread): the
        # shortest schedules of radices that divide its width
        for w in (12, 20):
            if n % w == 0:
                mixed = _factorisations(n, [q for q in (20, 12, 10, 6, 5, 4, 3, 2) if w % q == 0], 4)
                if mixed:
                    mnm = min(len(s) for s in mixed)
                    scheds += [s for s in mixed if len(s) == mnm and s not in scheds][:3]
    tiles = (0, 4, 8, 16, 32) if axis == 0 else (0, 8, 16, 32)
    return [(s, t) for s, t in itertools.product(scheds, tiles)]


def _time_plan(scen, axis: Optional[int], sched: Optional[List[int]], tile: int, steps: int) -> Optional[Dict[str, float]]:
    """ms a step of each kernel class, with a schedule forced on one axis (axis None:
    the library's defaults); None for a schedule that does not fit."""
    from . import _abi as A
    from .simulation import Simulation
    try:
        sim = Simulation(scen, tune=False)
        if axis is not None:
            sim.set_plan(axis, sched, tile)
    except A.KwError:
        return None
    sim.step(2)
    sim.synchronize()
    sim.stats()
    sim.profile(True)
    base = sim.stats()["classes"]
    sim.step(steps)
    st = sim.stats()["classes"]
    sim.profile(False)
    sim.close()
    return {c: (st[c]["ms"] - base[c]["ms"]) / steps for c in st}


def _tune(scen, axes, steps: int, verbose: bool) -> Dict[int, Dict]:
    """The cache entries of the axes: the fastest schedule of the engines, marked
    "forced" where the whole step is faster with it than with the library's
    defaults: the best of three timings of each in turn, by more than 2 % (the
    first timing on an idle card was 2.5 % slow at 256^3, the next two 0.5 % apart).
    An axis whose passes run on staged transforms by default is left there by an
    entry without the mark."""
    def step_ms(axis, sched, tile):
        return sum(_time_plan(scen, axis, sched, tile, steps).values())

    out = {}
    for axis in axes:
        n = lengths(scen.grid)[axis]
        best = None
        for sched, tile in candidates(axis, n):
            ms = _time_plan(scen, axis, sched, tile, steps)
            if ms is None:
                continue
            own = sum(ms[c] for c in AXIS_CLASSES[axis])
            if verbose:
                print("tune axis %d n=%d %-14s tile %2d: %.4f ms/step" % (axis, n, sched, tile, own),
                      flush=True)
            if best is None or own < best[2]:
                best = (sched, tile, own)
        if best is None:
            continue
        out[axis] = dict(radices=best[0], tile=best[1], ms=best[2])
        pairs = [(step_ms(None, None, 0), step_ms(axis, *best[:2])) for _ in range(3)]
        default, forced_ms = (min(p[i] for p in pairs) for i in (0, 1))
        if forced_ms < 0.98 * default:
            out[axis]["forced"] = True
        if verbose:
            print("tune axis %d: step %.4f ms with it, %.4f ms by default" % (axis, forced_ms, default), flush=True)
    return out


def tune(scen, axes=(0, 1, 2), steps: int = 4, verbose: bool = True, save: bool = True) -> Dict:
    """Time every candidate schedule for the requested axes of `scen` and
    record the fastest in the cache.  Returns {axis: (schedule, tile, ms)}."""
    cache = load_cache()
    arch = _arch()
    found = _tune(scen, axes, steps, verbose)
    if save:
        for axis, e in found.items():
            cache[key(axis, lengths(scen.grid)[axis], arch)] = e
        save_cache(cache)
    return {axis: (e["radices"], e["tile"], e["ms"]) for axis, e in found.items()}


def _entries(grid) -> Dict[int, Dict]:
    """Cached choices for the axes of `grid`: the user's cache first, then the table
    shipped with the package ({} when neither has an entry)."""
    arch = _arch()
    tables = (load_cache(), shipped_table(arch))
    out = {}
    for axis, n in enumerate(lengths(grid)):
        for tab in tables:
            e = tab.get(key(axis, n, arch))
            if e:
                out[axis] = e
                break
    return out


def lookup(grid) -> Dict[int, Tuple[List[int], int]]:
    """{axis: (schedule, tile)} of the cached choices for `grid`."""
    return {axis: (list(e["radices"]), int(e.get("tile", 0))) for axis, e in _entries(grid).items()}


def forced(grid) -> Set[int]:
    """Axes of `grid` whose cached schedule made the step faster than the library's
    defaults did: applied with kw_set_plan, the others as hints."""
    return {axis for axis, e in _entries(grid).items() if e.get("forced")}


def tune_table(sizes, steps: int = 3, out: Optional[str] = None, verbose: bool = True) -> Dict:
    """Tune every axis for each cubic size in `sizes` (for lengths above 256
    on a grid whose other two axes are 64 points, one axis at a time) and
    return {key: choice}; with `out`, also write it as JSON (the format of the
    shipped tables)."""
    from . import scenarios as sc
    arch = _arch()
    table = {}
    for n in sizes:
        if n <= 256:
            jobs = [(sc.small_case(n, n, n, seed=0, steps=8), (0, 1, 2))]
        else:
            jobs = []
            for axis in range(3):
                shape = [64, 64, 64]
                shape[axis] = n
                jobs.append((sc.small_case(*shape, seed=0, steps=8), (axis,)))
        for scen, axes in jobs:
            for axis, e in _tune(scen, axes, steps, verbose).items():
                table[key(axis, lengths(scen.grid)[axis], arch)] = dict(e, ms=round(e["ms"], 5))
            if verbose:
                print("tuned n=%d axes %s" % (n, axes), flush=True)
    if out:
        with open(out, "w") as fh:
            json.dump(table, fh, indent=1, sort_keys=True)
    return table


if __name__ == "__main__":
    import argparse
    ap = argparse.ArgumentParser(prog="python -m paper_1408_4675_amd.autotune")
    ap.add_argument("--sizes", type=int, nargs="+", default=[64, 96, 128, 160, 192, 256, 1024])
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--out", default=None, help="write the table here (JSON)")
    a = ap.parse_args()
    tune_table(a.sizes, a.steps, a.out)
