"""States outside the FP64 range in the passes: an infinite or overflowing K^mu in the root
solve, and pi~ whose square overflows in the regulator, give what IEEE quotients and roots give
(the CPU oracle's root solve and step, infinities included).  One cell in Cartesian coordinates:
no flux or source turns the values into NaN before the solve sees them."""
import numpy as np
import pytest

import oracle as O
from hydro_inputs import eos as EOS
from hydro_inputs import workloads as W
from tests import gpu_common as G

pytestmark = pytest.mark.gpu

INF = float("inf")


def _workload(T, pi=None):
    p = dict(nx=1, ny=1, ne=1, dx=0.3, dy=0.3, de=0.3, tau0=0.6, h=0.01, cartesian=1,
             etas=0.08 if pi is not None else 0.0, viscous=int(pi is not None))
    ic = None if pi is None else {"pi": np.array(pi, dtype=float).reshape(10, 1, 1, 1)}
    return W.Workload("one_cell", p, EOS.cached_synthetic_table(), 1, ic=ic,
                      T4=np.array(T, dtype=float).reshape(4, 1, 1, 1))


def _solves(wl, T, n):
    """(e, u~) of the last of n root solves of K = T, each from the e of the one before (the
    first, cold, is the initial state's), and the counters of all but the first."""
    o = O.Oracle(G.oracle_params(wl.params), eos=wl.eos)
    e, count = None, dict.fromkeys(("solves", "fallbacks", "nonconv", "clamps"), 0)
    for k in range(n):
        e, u, it, fl = o.con2prim(np.array(T), guess=e)
        if k:
            count["solves"] += int(it[0] > 0)
            count["fallbacks"] += int(fl[0] & O.C2P_FALLBACK != 0)
            count["nonconv"] += int(fl[0] & O.C2P_NONCONV != 0)
            count["clamps"] += int(fl[0] & O.C2P_CLAMP != 0)
    return [e[0], *u[0]], count


@pytest.mark.parametrize("tile", [-1, 0])
@pytest.mark.parametrize("T", [(1e200, 3e153, 0.0, 0.0), (1e200, 0.0, 0.0, 0.0),
                               (1e200, 1e100, 0.0, 0.0), (1e160, 1e153, 0.0, 0.0),
                               (1e160, 1e140, -1e150, 1.0)])
def test_root_solve(T, tile):
    """T~ does not change, so every pass solves K = T~."""
    print(f"[gpu-case] root solve of {T} tile {tile}", flush=True)
    wl = _workload(T)
    g = G.run_gpu(wl, 2, tile=tile)
    f, d = g.fields(), g.diag()
    want, count = _solves(wl, T, 5)
    np.testing.assert_allclose([f[k].item() for k in ("eps", "ux", "uy", "ue")], want, rtol=1e-13)
    assert [f[f"T{m}"].item() for m in range(4)] == list(T)
    assert {k: d[k] for k in count} == count and d["nans"] == d["vacuum"] == 0


@pytest.mark.parametrize("tile", [-1, 0])
@pytest.mark.parametrize("T", [(INF, 0.0, 0.0, 0.0), (INF, 2.0, -1.0, 0.5), (INF, INF, 0.0, 0.0),
                               (5.0, INF, 0.0, 0.0)])
def test_infinite_state(T, tile):
    """The predictor solves the infinite K; the corrector's T~' - T~ is NaN, hence vacuum."""
    print(f"[gpu-case] infinite {T} tile {tile}", flush=True)
    wl = _workload(T)
    g = G.run_gpu(wl, 1, tile=tile)
    f, d = g.fields(), g.diag()
    _, count = _solves(wl, T, 2)
    assert {k: d[k] for k in count} == count
    assert d["nans"] == d["vacuum"] == 1 and f["eps"].item() == 0.0


@pytest.mark.parametrize("tile", [-1, 0])
@pytest.mark.parametrize("E,big", [(10.0, 1e149), (10.0, 1e150), (10.0, 1e155), (10.0, 1e170),
                                   (1e160, 3e160), (1e160, 1e155), (1e200, 1e170),
                                   (1e160, 1e100)])
def test_regulator(E, big, tile):
    """A shear stress whose square overflows is scaled to zero, also next to an e whose square
    does; the cell keeps its e."""
    print(f"[gpu-case] regulator {E} {big} tile {tile}", flush=True)
    pi = np.zeros(10)
    pi[4], pi[7] = big, -big  # xx and yy: K is not touched
    wl = _workload((E, 0.1 * E if E < 1e100 else 0.0, 0.0, 0.0), pi)
    g, o = G.run_gpu(wl, 2, tile=tile), G.run_oracle(wl, 2)
    G.assert_parity(g.fields(), o.fields(), 1e-12, f"pi {big}")
    dg, do = g.diag(), o.diag()
    for k in ("solves", "clamps", "nans", "vacuum", "negative"):
        assert dg[k] == do[k], k
    assert dg["nans"] == dg["vacuum"] == 0
