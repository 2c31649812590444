"""Vacuum tiles are known by marks that each pass leaves for the next.  Setting the tile shape
again drops the marks, so a run that does so before every step tests the fields each time: it
has to give the same bits (fields, counters, diagnostic sums) as one that keeps them.  Every
tile shape (neighbourhoods of one and two tiles per axis, the single-row tile whose
neighbours do not fit a wave), ideal / viscous / lambda_1 / bulk and baryon / mixed, without
the regulator (no marks are used), matter that spreads into marked tiles, quiet skipping,
graph replay, a change of shape, a new initial state, and a group."""
import numpy as np
import pytest

from hydro_inputs import workloads as W
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


def _same(a, b, label):
    fa, fb = a.fields(), b.fields()
    for k in fa:
        np.testing.assert_array_equal(fa[k], fb[k], err_msg=f"{label} {k}")
    assert a.diag() == b.diag(), label


def _workload(kind, n=(43, 37, 21), seed=5):
    kw = dict(nx=n[0], ny=n[1], ne=n[2], dx=0.9, dy=0.9, de=0.7, steps=8, seed=seed)
    return W.hotspots_bulk(**kw) if kind == "bulk" else W.hotspots_viscous(**kw)


def _start(wl, tile, **over):
    import paper_1802_04449_amd as K
    h = K.Hydro(tile=tile, **{**wl.params, **over})
    h.set_eos(wl.eos)
    h.set_initial(wl.ic)
    return h


def _step_unmarked(h, tile, n):
    import paper_1802_04449_amd as K
    for _ in range(n):
        K.ktmi_set_tile(h.h, tile)
        h.step(1)


OVER = {"ideal": {"viscous": 0}, "lambda1": {"lambda1_hat": -10.0}, "mixed": {"precision": 1},
        "no_regulator": {"pi_reg": 0.0}, "fast": {"h": 0.2}}


@pytest.mark.parametrize("tile", [0, 1, 2, 3, 4, 5])
@pytest.mark.parametrize("kind", ["ideal", "viscous", "lambda1", "bulk", "mixed", "no_regulator",
                                  "fast"])
def test_marks_change_nothing(kind, tile):
    print(f"[gpu-case] marks {kind} tile {tile}", flush=True)
    wl = _workload(kind)
    a, b = (_start(wl, tile, **OVER.get(kind, {})) for _ in range(2))
    a.step(6)
    _step_unmarked(b, tile, 6)
    _same(a, b, f"{kind} tile {tile}")
    assert a.diag()["vacuum"] > 0


@pytest.mark.parametrize("n", [(61, 59, 1), (200, 1, 3), (1, 90, 40)])
def test_thin_grids(n):
    wl = _workload("viscous", n)
    for tile in (0, 4):
        a, b = (_start(wl, tile) for _ in range(2))
        a.step(5)
        _step_unmarked(b, tile, 5)
        _same(a, b, f"{n} tile {tile}")


@pytest.mark.parametrize("kind", ["viscous", "bulk", "ideal"])
def test_shape_change_quiet_graph_and_new_state(kind):
    import torch

    import paper_1802_04449_amd as K
    wl, wl2 = _workload(kind), _workload(kind, seed=9)
    over = OVER.get(kind, {})
    wl2.ic["eps"] = np.roll(wl2.ic["eps"], 11, axis=0)  # matter where the first state had none
    runs = []
    for keep in (True, False):
        st = torch.cuda.Stream()
        h = K.Hydro(stream=st, tile=0, **{**wl.params, **over})
        h.set_eos(wl.eos)
        h.set_initial(wl.ic)

        def go(n, tile):
            if keep:
                h.step(n)
            else:
                _step_unmarked(h, tile, n)
        go(3, 0)
        K.ktmi_set_tile(h.h, 2)
        go(2, 2)
        K.ktmi_set_tile(h.h, 0)
        if keep:
            h.set_graph(True)
        for _ in range(4):
            go(1, 0)
            h.diag()  # eager work between the replays
        if keep:
            h.set_graph(False)
        K.ktmi_set_quiet_skip(h.h, 1 if keep else 0)
        go(3, 0)
        K.ktmi_set_quiet_skip(h.h, 0)
        go(2, 0)
        h.set_initial(wl2.ic)
        go(4, 0)
        runs.append(h)
    _same(*runs, kind)


def test_group():
    import paper_1802_04449_amd as K
    wls = [_workload("viscous", (43, 37, 21), 5), _workload("viscous", (31, 45, 17), 6),
           _workload("bulk", (33, 29, 21), 7)]
    hs = [_start(wl, 0) for wl in wls]
    alone = [_start(wl, 0) for wl in wls]
    grp = K.Group(hs)
    grp.step(3)
    for h, b in zip(hs, alone):
        h.step(1)  # and alone in between
        _step_unmarked(b, 0, 4)
    grp.step(2)
    for h, b, wl in zip(hs, alone, wls):
        _step_unmarked(b, 0, 2)
        _same(h, b, wl.name)
