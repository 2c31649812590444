"""The large-grid FP64 kernels on small grids: there the automatic tile runs events on kernels
of their own, so these take explicit tiles.  Quiet skipping over long runs, in which the flags
share their words with the vacuum marks and sleeping tiles carry theirs along; parity with the
oracle; and events with vacuum against the small-event kernels, which use no marks at all (a
wrong mark or neighbour would show there, also one of e' that lives within a step)."""
import numpy as np
import pytest

from hydro_inputs import workloads as W

from . import gpu_common as G

pytestmark = pytest.mark.gpu

SUMS = ("sum_Ttt", "geo_src", "newton_mean")


def _start(wl, tile, quiet=False, stream=None, **over):
    import paper_1802_04449_amd as K
    h = K.Hydro(stream=stream, tile=tile, **{**wl.params, **over})
    h.set_eos(wl.eos)
    h.set_quiet_skip(quiet)
    h.set_initial(wl.ic)
    return h


def _same(a, b, label, sums=True):
    fa, fb = a.fields(), b.fields()
    for k in fa:
        np.testing.assert_array_equal(fa[k], fb[k], err_msg=f"{label} {k}")
    da, db = a.diag(), b.diag()
    skip = () if sums else SUMS
    assert {k: da[k] for k in da if k not in skip} == {k: db[k] for k in db if k not in skip}, label
    for k in skip:  # the same terms, folded tile by tile
        assert da[k] == pytest.approx(db[k], rel=1e-12, abs=1e-300), (label, k)


KINDS = {"ideal": {"viscous": 0, "etas": 0.0}, "viscous": {}, "cartesian": {"cartesian": 1},
         "lambda1": {"lambda1_hat": -10.0, "taupi_coef": 7.5}, "bulk": {}, "mixed": {"precision": 1}}


def _workload(kind, n, steps, seed, dx):
    kw = dict(nx=n[0], ny=n[1], ne=n[2], dx=dx, dy=dx, de=0.5, steps=steps, seed=seed)
    return W.hotspots_bulk(**kw) if kind == "bulk" else W.hotspots_viscous(**kw)


@pytest.mark.parametrize("tile", [0, 2])
@pytest.mark.parametrize("kind", list(KINDS))
def test_quiet_skip(kind, tile):
    """120 steps: matter crosses several tile boundaries and wakes sleeping tiles."""
    import paper_1802_04449_amd as K
    print(f"[gpu-case] large-grid quiet skip {kind} tile {tile}", flush=True)
    wl = _workload(kind, (61, 61, 9), 120, 31, 0.35)
    a, b = (_start(wl, tile, on, **KINDS[kind]) for on in (False, True))
    slept = []
    for n in (1, 4, 35, 80):
        a.step(n)
        b.step(n)
        q, total = K.ktmi_quiet_tiles(b.h)
        slept.append(q)
    _same(a, b, f"{kind} tile {tile}")
    assert 0 < q < total and slept[-1] < max(slept), slept  # some slept, some were woken


def test_quiet_skip_grouped_graph():
    import torch

    import paper_1802_04449_amd as K
    print("[gpu-case] large-grid quiet skip group graph", flush=True)
    st = torch.cuda.Stream()
    evs = [(_workload(k, n, 40, s, 0.5), t, KINDS[k])
           for k, n, s, t in (("viscous", (45, 43, 9), 70, 0), ("ideal", (41, 41, 17), 71, 2),
                              ("bulk", (43, 45, 7), 72, 0), ("viscous", (47, 41, 11), 73, 0))]
    hs = [_start(wl, t, True, st, **over) for wl, t, over in evs]
    grp = K.Group(hs)
    grp.set_graph(True)
    for n in (3, 12, 25):
        grp.step(n)
        [h.read("eps").sum() for h in hs]  # eager work between the replays
        torch.cuda.synchronize()
    for (wl, t, over), h in zip(evs, hs):
        q, total = K.ktmi_quiet_tiles(h.h)
        assert 0 < q < total
        ref = _start(wl, t, False, **over)
        ref.step(40)
        _same(h, ref, wl.name)


@pytest.mark.parametrize("kind", [k for k in KINDS if k != "mixed"])
def test_matches_the_kernels_without_marks(kind):
    """30 steps with vacuum against the small-event kernels, bit for bit."""
    import paper_1802_04449_amd as K
    print(f"[gpu-case] marks against none {kind}", flush=True)
    n = (43, 37, 21)
    wl = _workload(kind, n, 30, 5, 0.9)
    ref = _start(wl, -1, **KINDS[kind])
    ref.step(30)
    assert K.ktmi_quiet_tiles(ref.h)[1] == 11 * 10 * 7  # 4 x 4 x 3 cells each
    assert 0 < ref.diag()["vacuum"] < 43 * 37 * 21
    for tile in range(K.ktmi_tile_count()):
        h = _start(wl, tile, **KINDS[kind])
        h.step(30)
        _same(h, ref, f"{kind} tile {tile}", sums=False)


@pytest.mark.parametrize("tile", [0, 1, 2, 3])
@pytest.mark.parametrize("kind", [k for k in KINDS if k != "mixed"])
def test_matches_the_oracle(kind, tile):
    print(f"[gpu-case] large-grid parity {kind} tile {tile}", flush=True)
    wl = _workload(kind, (37, 33, 13), 12, 5, 0.45)
    g, o = G.run_gpu(wl, 12, tile=tile, **KINDS[kind]), G.run_oracle(wl, 12, **KINDS[kind])
    G.assert_parity(g.fields(), o.fields(), 1e-12, f"{kind} tile {tile}")


@pytest.mark.parametrize("n", [(61, 59, 1), (5, 1, 4), (1, 90, 5), (9, 4, 3)])
def test_thin_grids_match_the_kernels_without_marks(n):
    import paper_1802_04449_amd as K
    for kind in ("ideal", "viscous", "bulk"):
        wl = _workload(kind, n, 15, 9, 0.9)
        ref = _start(wl, -1, **KINDS[kind])
        ref.step(15)
        for tile in range(K.ktmi_tile_count()):
            h = _start(wl, tile, **KINDS[kind])
            h.step(15)
            _same(h, ref, f"{kind} {n} tile {tile}", sums=False)
