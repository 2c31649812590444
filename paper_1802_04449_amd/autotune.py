"""Tile-shape autotuner: times every workgroup tile shape of the stencil kernels on
a given grid through the C ABI and keeps the fastest.

The library's default (fewest padded thread slots, coalescing-aware) is a
reasonable start; the best shape depends on the grid's extents, the vacuum
fraction and the mode, so it is measured.  Where the automatic setting runs a
small event on kernels of its own, which no explicit shape selects, it is timed
too and kept if it wins.  Results are cached per grid, physics, precision and
guess mode in a JSON file next to this module.
"""
from __future__ import annotations

import json
import os
import time

from . import (KtmiError, ktmi_get_tile, ktmi_set_tile, ktmi_tile_count, ktmi_tile_shape)

CACHE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "autotune_cache.json")


KERNELS = 2  # raised when kernels change enough to move the best shape


def _key(hydro, automatic) -> str:
    d = hydro.desc
    return (f"k{KERNELS}:{d.nx}x{d.ny}x{d.ne}:v{d.viscous}:c{d.cartesian}:p{d.precision}"
            f":l{int(d.lambda1_hat != 0.0)}:z{int(d.zetas > 0.0)}:b{d.baryon}:g{d.guess}"
            f":a{int(automatic)}")


def _time(hydro, steps, repeats):
    """Best of `repeats` times per step in ms (after one step for the first launch)."""
    torch = hydro.torch
    best = float("inf")
    hydro.step(1)
    for _ in range(repeats):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        hydro.step(steps)
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t0) / steps * 1e3)
    return best


def tune(hydro, steps: int = 3, repeats: int = 2, use_cache: bool = True, verbose=False,
         automatic: bool = True):
    """Time `steps` steps per tile shape (best of `repeats`) on hydro's current state
    and select the fastest.  The state advances during tuning, so call it before the
    run of interest (or on a throwaway copy).  Returns (tile, {tile: ms_per_step}).

    The automatic setting, which may run on the small-event kernels, is one of the candidates,
    under the index of its shape (ktmi_get_tile): if it wins, that index is returned and the
    handle is left automatic.  automatic = False leaves it out, for events that are to be
    stepped with the returned tile in a group large enough to fill the GPU."""
    key = _key(hydro, automatic)
    cache = {}
    if use_cache and os.path.exists(CACHE):
        try:
            cache = json.load(open(CACHE))
        except (OSError, ValueError):
            cache = {}
    if use_cache and key in cache:
        ktmi_set_tile(hydro.h, int(cache[key]["set"]))
        return int(cache[key]["tile"]), cache[key]["ms"]
    times = {}
    own = None  # index of the automatic shape, if the automatic setting beats it
    if automatic:
        ktmi_set_tile(hydro.h, -1)
        auto, ms = ktmi_get_tile(hydro.h), _time(hydro, steps, repeats)
    for t in range(ktmi_tile_count()):
        try:
            ktmi_set_tile(hydro.h, t)
        except KtmiError:
            continue
        times[t] = _time(hydro, steps, repeats)
        if automatic and t == auto and ms < times[t]:
            own, times[t] = t, ms
        if verbose:
            print(f"tile {t} {ktmi_tile_shape(t)}{' (automatic)' if own == t else ''}: "
                  f"{times[t]:.3f} ms/step", flush=True)
    t = min(times, key=times.get)
    ktmi_set_tile(hydro.h, -1 if t == own else t)
    if use_cache:
        cache[key] = {"tile": t, "set": -1 if t == own else t, "shape": list(ktmi_tile_shape(t)),
                      "ms": {str(k): v for k, v in times.items()}}
        try:
            json.dump(cache, open(CACHE, "w"), indent=1)
        except OSError:
            pass
    return t, times


def current_shape(hydro):
    return ktmi_tile_shape(ktmi_get_tile(hydro.h))
