"""Small events with an automatic tile run on kernels of their own (about 50 cells per
workgroup, one wave per axis); any explicit tile keeps the large-grid kernels.  Fields and
counters are equal bit for bit, the diagnostic sums up to their order; grids with remainders
along every axis, single-cell axes, ideal / viscous / lambda_1 / bulk and baryon (mixed
precision keeps the large-grid kernels), with and without vacuum, graph replay, and the
switch between the two kinds of kernel in the middle of a run."""
import numpy as np
import pytest

from hydro_inputs import workloads as W
from tests import gpu_common as G

pytestmark = pytest.mark.gpu

COUNTS = ("step", "eps_max", "max_cfl", "newton_max", "solves", "fallbacks", "nonconv", "nans",
          "vacuum", "clamps", "negative", "errors")


def _same(a, b, label):
    fa, fb = a.fields(), b.fields()
    for k in fa:
        np.testing.assert_array_equal(fa[k], fb[k], err_msg=f"{label} {k}")
    da, db = a.diag(), b.diag()
    assert {k: da[k] for k in COUNTS} == {k: db[k] for k in COUNTS}, label
    for k in ("sum_Ttt", "geo_src", "newton_mean"):  # the same terms in another order
        assert da[k] == pytest.approx(db[k], rel=1e-12, abs=1e-300), (label, k)


@pytest.mark.parametrize("kind", ["ideal", "viscous", "lambda1", "bulk", "mixed", "mixed_ideal"])
@pytest.mark.parametrize("n", [(23, 21, 7), (16, 14, 1), (17, 13, 1), (9, 4, 3), (5, 1, 4), (1, 6, 2),
                               (7, 1, 1)])
def test_equals_large_grid_kernels(kind, n):
    nx, ny, ne = n
    print(f"[gpu-case] small event {kind} {n}", flush=True)
    kw = dict(nx=nx, ny=ny, ne=ne, dx=0.5, dy=0.5, de=0.5, steps=5, seed=11)
    wl = W.hotspots_bulk(**kw) if kind == "bulk" else W.hotspots_viscous(**kw)
    over = {}
    if kind.endswith("ideal"):
        over["viscous"] = 0
    if kind == "lambda1":
        over["lambda1_hat"] = -10.0
    if kind.startswith("mixed"):
        over["precision"] = 1
    _same(G.run_gpu(wl, 5, tile=-1, **over), G.run_gpu(wl, 5, tile=0, **over), f"{kind} {n}")


def test_dense_conformal_and_conserved():
    for wl in (W.gubser_ideal_33(), W.hotspots_minijets(nx=27, ny=25, ne=5, dx=0.4, dy=0.4, de=0.5)):
        _same(G.run_gpu(wl, 6, tile=-1), G.run_gpu(wl, 6, tile=2), wl.name)


def test_switching_and_graph():
    import torch

    import paper_1802_04449_amd as K
    wl = W.hotspots_viscous(nx=33, ny=31, ne=5, dx=0.4, dy=0.4, de=0.5, seed=3)
    st = torch.cuda.Stream()
    runs = []
    for auto in (True, False):
        g = K.Hydro(stream=st, tile=-1 if auto else 0, **wl.params)
        g.set_eos(wl.eos)
        g.set_initial(wl.ic)
        g.step(2)
        if auto:
            K.ktmi_set_tile(g.h, 1)      # large-grid kernels
            g.step(1)
            K.ktmi_set_tile(g.h, -1)     # small-event kernels again
            g.set_graph(True)
            for _ in range(3):           # replays with eager work between
                g.step(1)
                g.read("eps").sum()
                torch.cuda.synchronize()
            g.set_graph(False)
            g.set_quiet_skip(True)       # quiet tiles: large-grid kernels
            g.step(1)
            g.set_quiet_skip(False)
            K.Group([g]).step(1)         # groups too
            g.step(1)
        else:
            g.step(7)
        runs.append(g)
    _same(runs[0], runs[1], "switching")
