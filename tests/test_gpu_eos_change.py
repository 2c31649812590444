"""A new EoS table on a live handle.  While P(0) != 0 the regulator leaves pi~ in vacuum cells;
once a table with P(0) = 0 is set, the passes take pi~ of a vacuum tile for zero.  What the
steps before have marked must not stand for that: the run equals one whose tile shape is set
again before every step, which clears the marks and tests the fields each time, and one on the
small-event kernels, which use none.

The states are rows of cells, vacuum on the left, a few cells just over the energy cutoff (they
fall below it, with pi~ in the vacuum next to them, and come back once pi~ is gone), dilute
matter on the right; with the first two seeds stale pi~ reaches the fields."""
import numpy as np
import pytest

from hydro_inputs import eos as EOS

pytestmark = pytest.mark.gpu


def _run(seed, steps, again, tile=1):
    import paper_1802_04449_amd as K
    rng = np.random.default_rng(seed)
    nx, t = 40, EOS.cached_synthetic_table()
    p0 = 10.0 ** rng.uniform(-8, -6)
    s, w = int(rng.integers(14, 24)), int(rng.integers(4, 9))
    e = np.zeros((nx, 1, 1))
    e[s:] = 1.0001e-7
    e[s + w:] = 10.0 ** rng.uniform(-6, -3)
    pi = rng.standard_normal((10, nx, 1, 1)) * (e + p0) * 10.0 ** rng.uniform(-0.7, 0.3) * (e > 0)
    u = rng.normal(0.0, 0.3, (3, nx, 1, 1)) * (e > 0)
    h = K.Hydro(nx=nx, ny=1, ne=1, dx=0.3, dy=0.3, de=0.3, tau0=0.6, h=0.01, etas=0.08, viscous=1,
                zetas=0.04, taubulk_coef=5.0, baryon=1, tile=tile)
    K.ktmi_set_eos_table(h.h, t.eps0, t.deps, np.array(t.P) + p0, t.T, t.cs2)
    h.set_initial(dict(eps=e, ux=u[0], uy=u[1], ue=u[2], pi=pi, Pi=np.zeros_like(e), nb=0.1 * (e > 0)))
    for n in range(steps):
        if n == 2:
            K.ktmi_set_eos_table(h.h, t.eps0, t.deps, t.P, t.T, t.cs2)
        if again:
            K.ktmi_set_tile(h.h, tile)
        h.step(1)
    return h.fields()


@pytest.mark.parametrize("seed", [911, 1826, 3])
def test_table_without_vacuum_pressure_follows_one_with_it(seed):
    print(f"[gpu-case] EoS change {seed}", flush=True)
    a, b, c = _run(seed, 5, False), _run(seed, 5, True), _run(seed, 5, False, tile=-1)
    for k in a:
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)
        np.testing.assert_array_equal(a[k], c[k], err_msg=k)
