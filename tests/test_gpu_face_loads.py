"""Face states looked up in the EoS table in pairs: a table that ends inside the event's
energy range, so that some waves have lanes past its end, on grids with and without vacuum
(waves that need pi~'s masks and waves that do not), ideal / viscous / bulk and baryon, on
the kernels of small and of large events.  Tolerance: the 1e-12 of every FP64 comparison
against the oracle."""
import dataclasses

import pytest

from hydro_inputs import workloads as W
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


def _cut(table, e_last):
    n = int((e_last - table.eps0) / table.deps) + 1
    return dataclasses.replace(table, P=table.P[:n].copy(), T=table.T[:n].copy(),
                               cs2=table.cs2[:n].copy())


@pytest.mark.parametrize("tile", [-1, 0])
@pytest.mark.parametrize("kind", ["ideal", "viscous", "bulk", "dense"])
@pytest.mark.parametrize("rows_to", [0.4, 20.0, 1e9])
def test_table_end_inside_the_event(rows_to, kind, tile):
    print(f"[gpu-case] table end {rows_to} {kind} tile {tile}", flush=True)
    d = 0.4 if kind == "dense" else 0.8  # hotspots: vacuum around the disk
    kw = dict(nx=27, ny=25, ne=9, dx=d, dy=d, de=0.5, steps=4)
    if kind == "bulk":
        wl = W.hotspots_bulk(seed=4, **kw)
    elif kind == "dense":
        wl = W.gubser_dense_viscous(**kw)
    else:
        wl = W.hotspots_viscous(seed=4, **kw)
    over = {"viscous": 0} if kind == "ideal" else {}
    wl.eos = _cut(wl.eos, min(rows_to, wl.eos.eps0 + wl.eos.deps * (len(wl.eos.P) - 1)))
    g, o = G.run_gpu(wl, 4, tile=tile, **over), G.run_oracle(wl, 4, **over)
    G.assert_parity(g.fields(), o.fields(), 1e-12, f"{wl.name} {rows_to} {kind} {tile}")
