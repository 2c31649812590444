"""At most 128 events of one tile shape, precision and mode in a group.  Small events keep to that
limit by the shape of their grid, not by the few shapes of their own kernels: a group that the
shapes allow is made, and one event more of a shape is refused."""
import pytest

from hydro_inputs import workloads as W

pytestmark = pytest.mark.gpu


def test_limit_is_per_shape_of_the_grid():
    import torch

    import paper_1802_04449_amd as K
    print("[gpu-case] group limit", flush=True)
    st = torch.cuda.Stream()
    wls = [W.hotspots_viscous(nx=8, ny=8, ne=ne, dx=1.5, dy=1.5, de=0.5, seed=3) for ne in (16, 8)]

    def start(wl):
        h = K.Hydro(stream=st, **wl.params)
        h.set_eos(wl.eos)
        h.set_initial(wl.ic)
        return h

    hs = [[start(wl) for _ in range(128)] for wl in wls]
    shapes = {K.ktmi_get_tile(h[0].h) for h in hs}
    assert len(shapes) == 2
    grp = K.Group(hs[0] + hs[1])  # 256 events, 128 of each shape
    grp.step(3)
    grp.set_graph(True)
    grp.step(2)
    for wl, members in zip(wls, hs):
        ref = start(wl)
        ref.step(5)
        a, d = ref.fields(), ref.diag()
        for h in (members[0], members[1], members[127]):
            b = h.fields()
            for k in a:
                assert (a[k] == b[k]).all(), k
            assert h.diag()["vacuum"] == d["vacuum"] and h.diag()["solves"] == d["solves"]
    with pytest.raises(K.KtmiError, match="max 128"):
        K.Group(hs[0] + [start(wls[0])])
