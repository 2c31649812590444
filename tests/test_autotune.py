"""What the autotuner chooses: the automatic setting (which may run a small event on kernels of
its own) is a candidate and is kept when it wins; a cached choice is set again; results of other
physics or of other kernels are not reused."""
import types

import pytest

from hydro_inputs import workloads as W


def _fake(monkeypatch, tmp_path, ms, **over):
    """A handle without a device, and times per tile setting (-1: automatic) for it."""
    import paper_1802_04449_amd as K
    from paper_1802_04449_amd import autotune
    d = K.ktmi_desc_default()
    for k, v in {**dict(nx=41, ny=37, ne=13, dx=0.3, dy=0.3, de=0.3, tau0=0.6, h=0.01, etas=0.08,
                        viscous=1), **over}.items():
        setattr(d, k, v)
    hydro = types.SimpleNamespace(h=K.ktmi_create(d), desc=d)
    state = {"set": -1}

    def set_tile(h, t):
        state["set"] = t
        K.ktmi_set_tile(h, t)

    monkeypatch.setattr(autotune, "ktmi_set_tile", set_tile)
    monkeypatch.setattr(autotune, "_time", lambda *_: ms[state["set"]])
    monkeypatch.setattr(autotune, "CACHE", str(tmp_path / "cache.json"))
    return hydro, state


def test_automatic_setting_is_kept_when_it_wins(monkeypatch, tmp_path):
    import paper_1802_04449_amd as K
    from paper_1802_04449_amd import autotune
    ms = {t: 2.0 + 0.1 * t for t in range(K.ktmi_tile_count())}
    for auto_ms, wins in ((1.0, True), (1.95, True), (2.05, False), (9.0, False)):
        for sub in ("a", "b"):
            (tmp_path / f"{auto_ms}{sub}").mkdir()
        hydro, state = _fake(monkeypatch, tmp_path / f"{auto_ms}a", {-1: auto_ms, **ms})
        K.ktmi_set_tile(hydro.h, -1)
        shape = K.ktmi_get_tile(hydro.h)
        for again in range(2):  # measured, then from the cache
            t, times = autotune.tune(hydro)
            assert state["set"] == (-1 if wins else 0)
            assert t == K.ktmi_get_tile(hydro.h) == (shape if wins else 0)
            assert len(times) == K.ktmi_tile_count() and min(times.values()) == (auto_ms if wins else 2.0)
        # left out on request: the fastest explicit shape
        t, times = autotune.tune(hydro, automatic=False)
        assert t == state["set"] == 0 and min(times.values()) == 2.0
        K.ktmi_destroy(hydro.h)


def test_cache_tells_physics_and_kernels_apart(monkeypatch, tmp_path):
    import paper_1802_04449_amd as K
    from paper_1802_04449_amd import autotune
    n = K.ktmi_tile_count()
    first = {t: 1.0 + (t != 1) for t in range(-1, n)}
    other = {t: 1.0 + (t != 3) for t in range(-1, n)}
    hydro, _ = _fake(monkeypatch, tmp_path, first)
    assert autotune.tune(hydro)[0] == 1
    for over in (dict(lambda1_hat=-10.0), dict(zetas=0.04), dict(baryon=1), dict(precision=1),
                 dict(guess=K.KTMI_GUESS_COLD)):
        h2, _ = _fake(monkeypatch, tmp_path, other, **over)
        assert autotune.tune(h2)[0] == 3, over
        K.ktmi_destroy(h2.h)
    _fake(monkeypatch, tmp_path, other)
    assert autotune.tune(hydro)[0] == 1  # its own entry
    monkeypatch.setattr(autotune, "KERNELS", autotune.KERNELS + 1)
    assert autotune.tune(hydro)[0] == 3
    K.ktmi_destroy(hydro.h)


@pytest.mark.gpu
def test_tuned_small_event_keeps_its_kernels():
    """On 151x151x1 hotspots the small-event kernels take about 0.6 of the fastest shape."""
    import paper_1802_04449_amd as K
    from paper_1802_04449_amd import autotune
    print("[gpu-case] autotune 151x151x1", flush=True)
    wl = W.hotspots_viscous(nx=151, ny=151, ne=1, dx=0.16, dy=0.16, de=0.3, steps=4, seed=3)
    h = K.Hydro(**wl.params)
    h.set_eos(wl.eos)
    h.set_initial(wl.ic)
    t, times = autotune.tune(h, steps=10, repeats=3, use_cache=False)
    assert t == K.ktmi_get_tile(h.h) and times[t] == min(times.values())
    h.step(1)
    assert K.ktmi_quiet_tiles(h.h)[1] == 19 * 22  # tiles of 8 x 7 cells
