"""Freeze-out surface on random slices (every tetrahedron case, values equal to e_f among
them) over grid shapes: spans of hypercubes that cross rows and planes, axes of one and two
cells, runs of cells that just fit the workgroup's LDS and that do not.  Against the CPU
oracle: the same hypercubes in the same order, records to 1e-12 of each column's scale (the
same expressions in the same order)."""
import numpy as np
import pytest

import oracle as O
from hydro_inputs import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(9, 8, 65), (70, 66, 2), (2, 2, 4099), (1, 50, 60), (60, 1, 30),
                                   (1, 1, 9000), (130, 90, 1), (2, 5, 2), (2100, 2, 2),
                                   (2, 3, 14000), (3, 2, 20000)])
def test_random_slices(shape):
    import torch

    import paper_1802_04449_amd as K
    print(f"[gpu-case] surface shape {shape}", flush=True)
    rng = np.random.default_rng(shape[0] * 7 + shape[2])
    nx, ny, ne = shape
    A, B = (rng.uniform(0.0, 1.0, (4, nx, ny, ne)) for _ in range(2))
    ef = 0.75
    # smooth along eta (so that hypercubes of every kind occur), some values equal to e_f
    for S in (A, B):
        S[0] = np.round(0.5 * (S[0] + np.roll(S[0], 1, axis=2)) * 64) / 64
        S[0][rng.random((nx, ny, ne)) < 0.3] = ef
    wl = W.gubser_ideal_33()
    h = K.Hydro(**{**wl.params, "nx": nx, "ny": ny, "ne": ne})
    a, b = (torch.tensor(S, device="cuda") for S in (A, B))
    cap = (max(nx, 2) - 1) * (max(ny, 2) - 1) * (max(ne, 2) - 1)
    got = h.surface(a, 1.3, b, 1.35, ef, capacity=cap).cpu().numpy()
    p = wl.params
    ref = O.surface(shape, (p["dx"], p["dy"], p["de"]), A, 1.3, B, 1.35, ef)
    assert got.shape == ref.shape and len(ref) > 0
    np.testing.assert_array_equal(got[:, 0], ref[:, 0])
    scale = np.maximum(np.abs(ref).max(axis=0), 1e-300)
    assert (np.abs(got - ref) / scale).max() <= 1e-12
