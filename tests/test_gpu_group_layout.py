"""A member whose tile shape, guess mode or quiet skipping changes after its group was made:
the group goes on with the kernels it was made with, and the per-tile flags (vacuum marks, quiet
flags) that one tile layout leaves are never read in another.  Fields and counters equal a run
that steps with one tile alone."""
import numpy as np
import pytest

from hydro_inputs import workloads as W
from tests import gpu_common as G

pytestmark = pytest.mark.gpu

SUMS = ("sum_Ttt", "geo_src", "newton_mean")


def _same(a, b, label):
    fa, fb = a.fields(), b.fields()
    for k in fa:
        np.testing.assert_array_equal(fa[k], fb[k], err_msg=f"{label} {k}")
    da, db = a.diag(), b.diag()
    assert {k: da[k] for k in da if k not in SUMS} == {k: db[k] for k in db if k not in SUMS}, label
    for k in SUMS:  # the same terms, folded tile by tile
        assert da[k] == pytest.approx(db[k], rel=1e-12, abs=1e-300), (label, k)


def _start(wl, tile, **over):
    import paper_1802_04449_amd as K
    h = K.Hydro(tile=tile, **{**wl.params, **over})
    h.set_eos(wl.eos)
    h.set_initial(wl.ic)
    return h


@pytest.mark.parametrize("kind", ["ideal", "viscous", "bulk", "mixed"])
@pytest.mark.parametrize("tiles", [(0, 2), (2, 0), (-1, 0), (0, -1), (1, 3)])
def test_tile_changed_after_grouping(tiles, kind):
    import paper_1802_04449_amd as K
    print(f"[gpu-case] group layout {tiles} {kind}", flush=True)
    kw = dict(nx=43, ny=37, ne=21, dx=0.9, dy=0.9, de=0.7, steps=14, seed=5)
    wl = W.hotspots_bulk(**kw) if kind == "bulk" else W.hotspots_viscous(**kw)
    over = {"ideal": {"viscous": 0}, "mixed": {"precision": 1}}.get(kind, {})
    a, b = _start(wl, tiles[0], **over), _start(wl, 0, **over)
    grp = K.Group([a])
    grp.step(3)
    K.ktmi_set_tile(a.h, tiles[1])  # the group keeps its own tile
    grp.step(1)
    a.step(3)
    grp.step(2)
    a.step(1)
    grp.step(1)
    a.set_initial(wl.ic)  # marks of the first-step estimate in the handle's layout
    grp.step(2)
    b.step(11)
    b.set_initial(wl.ic)
    b.step(2)
    _same(a, b, f"{tiles} {kind}")


def test_guess_and_quiet_skip_changed_after_grouping():
    """The network runs on the large-grid kernels, a small event without it on its own ones;
    a group made without quiet skipping leaves no quiet flags."""
    import torch

    import paper_1802_04449_amd as K
    wl = W.hotspots_viscous(nx=61, ny=61, ne=9, dx=0.35, dy=0.35, de=0.5, steps=100, seed=31)
    rng = np.random.default_rng(0)
    prm = torch.as_tensor(0.1 * rng.standard_normal(K.ktmi_mlp_nparam()), dtype=torch.float32)
    a, b = _start(wl, -1), _start(wl, 0)
    grp = K.Group([a])
    grp.step(2)
    a.set_quiet_skip(True)
    for _ in range(3):
        a.step(3)
        grp.step(21)  # odd counts: both flag buffers
    a.step(2)
    a.set_quiet_skip(False)
    a.step(2)
    b.step(78)
    _same(a, b, "quiet skip")
    a.set_mlp(prm.cuda(), K.KTMI_MLP_FP32)  # large-grid kernels alone, small ones in the group
    b.set_mlp(prm.cuda(), K.KTMI_MLP_FP32)
    for h, grouped in ((a, grp.step), (b, b.step)):
        for _ in range(2):
            h.set_guess(K.KTMI_GUESS_MLP)
            h.step(3)
            if h is b:
                h.set_guess(K.KTMI_GUESS_PREV)
            grouped(3)  # made without the network
        h.set_guess(K.KTMI_GUESS_PREV)
        h.step(2)
    _same(a, b, "guess")
