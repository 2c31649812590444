"""Which events run on the small-event kernels: the tiles ktmi_quiet_tiles counts are those of
the last step's launches.  Alone by the tiles of the automatic shape and the faces it pads, in a
group also by what its small events fill together; fields and counters are the same either way,
the diagnostic sums up to their order."""
import numpy as np
import pytest

from hydro_inputs import workloads as W

pytestmark = pytest.mark.gpu

SUMS = ("sum_Ttt", "geo_src", "newton_mean")


def _start(n, tile=-1, kind="viscous", stream=None, seed=5):
    import paper_1802_04449_amd as K
    kw = dict(nx=n[0], ny=n[1], ne=n[2], dx=20.0 / n[0], dy=20.0 / n[0], de=0.4, steps=2, seed=seed)
    wl = W.hotspots_bulk(**kw) if kind == "bulk" else W.hotspots_viscous(**kw)
    h = K.Hydro(stream=stream, tile=tile, **{**wl.params, **({"viscous": 0} if kind == "ideal" else {})})
    h.set_eos(wl.eos)
    h.set_initial(wl.ic)
    return h


def _small_tiles(n):
    return -(-n[0] // 4) * -(-n[1] // 4) * -(-n[2] // 3) if n[2] > 1 else -(-n[0] // 8) * -(-n[1] // 7)


def _large_tiles(h, n):
    import paper_1802_04449_amd as K
    tx, ty, tz = K.ktmi_tile_shape(K.ktmi_get_tile(h.h))
    return -(-n[0] // tx) * -(-n[1] // ty) * -(-n[2] // tz)


def _same(a, b, label):
    fa, fb = a.fields(), b.fields()
    for k in fa:
        np.testing.assert_array_equal(fa[k], fb[k], err_msg=f"{label} {k}")
    da, db = a.diag(), b.diag()
    assert {k: da[k] for k in da if k not in SUMS} == {k: db[k] for k in db if k not in SUMS}, label
    for k in SUMS:
        assert da[k] == pytest.approx(db[k], rel=1e-12, abs=1e-300), (label, k)


@pytest.mark.parametrize("n,small", [((33, 33, 17), True), ((151, 151, 1), True), ((61, 61, 33), True),
                                     ((40, 40, 32), True), ((48, 48, 64), False),
                                     ((101, 101, 9), True), ((91, 89, 48), False),
                                     ((121, 121, 33), False), ((801, 700, 1), False)])
def test_alone(n, small):
    import paper_1802_04449_amd as K
    print(f"[gpu-case] route {n}", flush=True)
    h = _start(n)
    h.step(1)
    assert K.ktmi_quiet_tiles(h.h)[1] == (_small_tiles(n) if small else _large_tiles(h, n))
    for tile, prec in ((K.ktmi_get_tile(h.h), 0), (-1, 1)):  # explicit, mixed: never
        g = _start(n, tile) if prec == 0 else None
        if prec:
            wl = W.hotspots_viscous(nx=n[0], ny=n[1], ne=n[2], dx=20.0 / n[0], dy=20.0 / n[0], de=0.4)
            g = K.Hydro(tile=-1, **{**wl.params, "precision": 1})
            g.set_eos(wl.eos)
            g.set_initial(wl.ic)
        g.step(1)
        assert K.ktmi_quiet_tiles(g.h)[1] == _large_tiles(g, n)
        if prec == 0:
            _same(h, g, str(n))


@pytest.mark.parametrize("kind", ["ideal", "viscous", "bulk"])
def test_in_groups(kind):
    """Up to what fills the chip the members keep their kernels; beyond it those of more than
    one eta cell move to the large-grid ones.  Events of another mode do not count."""
    import torch

    import paper_1802_04449_amd as K
    print(f"[gpu-case] routes in groups {kind}", flush=True)
    n, flat = (45, 45, 65), (61, 61, 1)
    other = "viscous" if kind != "viscous" else "ideal"
    for nev, small in ((1, True), (12, False)):
        st = torch.cuda.Stream()
        hs = [_start(n, kind=kind, stream=st, seed=3 + k % 2) for k in range(nev)]
        extra = [_start(flat, kind=kind, stream=st), _start((33, 31, 9), kind=other, stream=st)]
        grp = K.Group(hs + extra)
        grp.step(3)
        for k, h in enumerate(hs):
            assert K.ktmi_quiet_tiles(h.h)[1] == (_small_tiles(n) if small else _large_tiles(h, n))
        assert K.ktmi_quiet_tiles(extra[0].h)[1] == _small_tiles(flat)
        assert K.ktmi_quiet_tiles(extra[1].h)[1] == _small_tiles((33, 31, 9))
        for h in hs[:2]:
            h.step(1)  # alone in between: on its own kernels
        grp.step(2)
        for k, h in enumerate(hs[:3]):
            alone = _start(n, kind=kind, seed=3 + k % 2)
            alone.step(6 if k < 2 else 5)
            _same(h, alone, f"{kind} {nev} {k}")
