"""The work that users of this package have it do, as cases that can be timed.

Each case is one whole use of a public entry point: an event evolved from its
initial state (`Hydro`: set_initial, step or step_until, snapshot, read, diag), a
batch of uneven events (`Group` under graph replay), the freeze-out surface
between two slices (`ktmi_surface`), the Cooper-Frye spectra of a surface
(`spectra`) and a training step of the learned root-solve guess
(`mlp.Trainer.step`).  Inputs are synthetic and made here from the seed alone:
Gaussian hotspots and Gubser profiles on the package's Milne grids, a smooth
crossover equation of state tabulated like the package's own (1555 rows), surface
records and fluid states of the ranges that such events give.

`exact` evaluates the same formulas in plain torch FP64 (no package code): the
Kurganov-Tadmor RK2 step with minmod reconstruction, the root solve, the shear,
bulk and baryon sources and the regulator; the Kuhn-triangulation surface; the
Cooper-Frye integral; the network's gradient by autograd and one Adam step.
"""
from __future__ import annotations

import itertools
import math
from types import SimpleNamespace

import numpy as np
import torch

HBARC = 0.1973269804  # GeV fm
C_SB = 47.5 * math.pi ** 2 / 30.0 / HBARC ** 3
F64 = torch.float64
DEV = "cuda"

# physics common to the package's configurations
TAU0, ETAS, EPS_CUT, THETA, PI_REG, TAUPI, ZETAS, TAUBULK = 0.6, 0.08, 1e-7, 1.8, 0.3, 5.0, 0.04, 5.0


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # the smallest events: an ideal conformal 33x33x17 Gubser run to its end, its
        # largest energy density looked at every 10 steps (launches and latency)
        dict(name="gubser_33", kind="evolve", ic="gubser", nx=33, ny=33, ne=17, dx=0.3, de=0.3,
             h=0.02, viscous=False, precision="fp64", bulk=False, steps=50, check=10),
        # boost-invariant (one eta cell) viscous events, the usual event-by-event scan
        dict(name="plane_151", kind="evolve", ic="hotspots", nx=151, ny=151, ne=1, dx=0.16, de=0.3,
             h=0.01, viscous=True, precision="fp64", bulk=False, steps=40, check=0),
        # the package's benchmark event: viscous, FP64, 82% of the grid vacuum at tau0
        dict(name="event_201", kind="evolve", ic="hotspots", nx=201, ny=201, ne=105, dx=0.16,
             de=0.3, h=0.01, viscous=True, precision="fp64", bulk=False, steps=10, check=0),
        # the same event in mixed precision
        dict(name="event_201_mixed", kind="evolve", ic="hotspots", nx=201, ny=201, ne=105, dx=0.16,
             de=0.3, h=0.01, viscous=True, precision="mixed", bulk=False, steps=10, check=0),
        # a smooth profile with no vacuum cell on a ragged grid: every cell at work
        dict(name="dense_101", kind="evolve", ic="gubser", nx=101, ny=99, ne=65, dx=0.16, de=0.3,
             h=0.01, viscous=True, precision="fp64", bulk=False, steps=10, check=0),
        # bulk pressure and baryon density transported as well
        dict(name="bulk_baryon_121", kind="evolve", ic="hotspots", nx=121, ny=121, ne=33, dx=0.2,
             de=0.4, h=0.01, viscous=True, precision="fp64", bulk=True, steps=10, check=5),
        # the largest single event
        dict(name="large_385", kind="evolve", ic="hotspots", nx=385, ny=385, ne=129, dx=0.08,
             de=0.15, h=0.005, viscous=True, precision="fp64", bulk=False, steps=3, check=0),
        # uneven events (ideal and viscous, one or more eta cells) stepped together
        dict(name="batch_8", kind="batch", steps=10, precision="fp64",
             events="101x33x0.08,151x1x0.08,117x65x0,131x33x0.16,201x1x0,109x33x0.08,125x65x0.16,"
                    "183x1x0.08"),
        # freeze-out surface between two slices with pi~
        dict(name="surface_201", kind="surface", nx=201, ny=201, ne=105, dx=0.16, de=0.3,
             with_pi=True, eps_f=0.3),
        # smooth spectra of eight species with delta f on the usual (Y, pT, phi) bins
        dict(name="spectra_8", kind="spectra", n=41660, ns=8, nY=41, npt=15, nphi=48, df=True),
        # one Adam step of the learned guess on the usual minibatch
        dict(name="train_8192", kind="train", batch=8192, mode="fp32"),
        # the gradient over a whole harvested state (and one Adam step)
        dict(name="train_1m", kind="train", batch=1000003, mode="bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges."""
    kind = rng.choice(["evolve"] * 6 + ["batch", "surface", "spectra", "train"])
    if kind == "evolve":
        ic = rng.choice(["hotspots", "hotspots", "gubser"])
        n, ne = _log_int(rng, 33, 241), rng.choice([1, _log_int(rng, 5, 105), _log_int(rng, 17, 105)])
        viscous = rng.random() < 0.8
        # bulk pressure and baryon density run in FP64 only
        bulk = viscous and rng.random() < 0.2
        mixed = not bulk and rng.random() < 0.25
        dx = rng.uniform(18.0, 32.0) / n if ic == "hotspots" else rng.uniform(9.0, 16.0) / n
        dx = min(max(dx, 0.08), 0.5)
        de = min(max(rng.uniform(8.0, 30.0) / ne, 0.15), 0.5)
        steps = max(3, min(50, int(4e7 / (n * n * ne))))
        return dict(kind="evolve", ic=ic, nx=n, ny=n + rng.randrange(-3, 4), ne=ne,
                    dx=round(dx, 4), de=round(de, 4),
                    h=round(min(0.01, 0.0625 * dx, 0.05 * de), 5), viscous=viscous,
                    precision="mixed" if mixed else "fp64", bulk=bulk, steps=steps,
                    check=rng.choice([0, 0, 5]))
    if kind == "batch":
        ev = []
        for _ in range(rng.randrange(2, 9)):
            ev.append("%dx%dx%s" % (rng.randrange(61, 182, 2), rng.choice([1, 17, 33, 65]),
                                    rng.choice(["0", "0.08", "0.16"])))
        return dict(kind="batch", steps=rng.randrange(5, 13),
                    precision=rng.choice(["fp64", "fp64", "mixed"]), events=",".join(ev))
    if kind == "surface":
        n, ne = _log_int(rng, 41, 221), rng.choice([1, _log_int(rng, 9, 105)])
        return dict(kind="surface", nx=n, ny=n + rng.randrange(-3, 4), ne=ne,
                    dx=round(min(max(28.0 / n, 0.12), 0.5), 4), de=0.3,
                    with_pi=rng.random() < 0.7, eps_f=round(rng.uniform(0.15, 0.6), 3))
    if kind == "spectra":
        n = _log_int(rng, 500, 40000)
        return dict(kind="spectra", n=n, ns=rng.randrange(1, 13), nY=rng.choice([1, 11, 21, 41]),
                    npt=rng.randrange(8, 21), nphi=rng.choice([1, 20, 24, 33, 48]),
                    df=rng.random() < 0.8)
    return dict(kind="train", batch=_log_int(rng, 1000, 1000000),
                mode=rng.choice(["fp32", "bf16"]))


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _table():
    """A smooth crossover EoS on 1555 rows, e_i = 0.04 i: cs2 = 1/3 - A exp(-ln^2(e/ec)/2)
    (0.14 at the dip), P = int cs2 de in closed form, T from dT/T = cs2 de/(e + P)."""
    if "t" in _CACHE:
        return _CACHE["t"]
    A, ec = 1.0 / 3.0 - 0.14, 0.45

    def cs2(e):
        return 1.0 / 3.0 - A * np.exp(-0.5 * np.log(e / ec) ** 2)

    def pressure(e):
        x = torch.as_tensor((np.log(e / ec) - 1.0) / math.sqrt(2.0), dtype=F64)
        dip = A * ec * math.exp(0.5) * math.sqrt(math.pi / 2.0)
        return e / 3.0 - dip * (1.0 + torch.erf(x).numpy())

    e = 0.04 * np.arange(1, 1555)
    # ln T = ln((e + P)/(4 C_SB/3))/4 - int_e^inf (3 cs2 - 1)/(4 (e + P)) de, trapezoids in ln e
    x = np.linspace(math.log(0.01), math.log(ec) + 12.0, 40001)
    ex = np.exp(x)
    g = (3.0 * cs2(ex) - 1.0) / (4.0 * (ex + pressure(ex))) * ex
    cum = np.concatenate([[0.0], np.cumsum(0.5 * (g[1:] + g[:-1]) * np.diff(x))])
    tail = cum[-1] - np.interp(np.log(e), x, cum)
    P = np.concatenate([[0.0], pressure(e)])
    T = np.concatenate([[0.0], (((e + P[1:]) / (4.0 * C_SB / 3.0)) ** 0.25) * np.exp(-tail)])
    c = np.concatenate([[1.0 / 3.0], cs2(e)])
    _CACHE["t"] = SimpleNamespace(eps0=0.0, deps=0.04, P=P, T=T, cs2=c)
    return _CACHE["t"]


_CACHE: dict = {}


def _axis(n, d):
    return (torch.arange(n, dtype=F64, device=DEV) - (n - 1) / 2.0) * d


def _woods_saxon(rng, n, R=6.5, a=0.5):
    out = []
    while len(out) < n:
        r = (R + 10.0 * a) * np.sqrt(rng.random(4 * n))
        ok = rng.random(4 * n) < 1.0 / (1.0 + np.exp((r - R) / a))
        phi = 2.0 * math.pi * rng.random(4 * n)
        out += list(np.stack([r * np.cos(phi), r * np.sin(phi)], axis=1)[ok])
    return np.array(out[:n])


def _hotspots(nx, ny, ne, dx, de, seed):
    """200 Gaussian hotspots (width 0.5 fm, Gamma(1) weights) in a Woods-Saxon disk times a
    plateau in eta, peak 55 GeV/fm^3, at rest."""
    rng = np.random.default_rng(seed)
    xy = torch.as_tensor(_woods_saxon(rng, 200), device=DEV)
    w = torch.as_tensor(rng.gamma(1.0, 1.0, 200), device=DEV)
    x, y, eta = _axis(nx, dx), _axis(ny, dx), _axis(ne, de)
    gx = torch.exp(-(x[None, :] - xy[:, :1]) ** 2 / 0.5) * w[:, None]
    gy = torch.exp(-(y[None, :] - xy[:, 1:]) ** 2 / 0.5)
    prof = torch.zeros(nx, ny, dtype=F64, device=DEV)
    for k in range(200):
        prof += gx[k, :, None] * gy[k, None, :]
    d = (eta.abs() - 2.0).clamp(min=0.0)
    eps = prof[:, :, None] * torch.exp(-d * d / (2.0 * 1.3 ** 2))[None, None, :]
    eps = (eps * (55.0 / eps.max())).contiguous()
    z = torch.zeros_like(eps)
    return dict(eps=eps, ux=z, uy=z.clone(), ue=z.clone())


def _gubser(nx, ny, ne, dx, de, tau, seed):
    """Ideal Gubser flow (q about 1/fm, peak T about 0.4 GeV at tau = 1/q)."""
    rng = np.random.default_rng(seed)
    q, Tp = 1.0 + 0.05 * rng.uniform(-1, 1), 0.4 + 0.02 * rng.uniform(-1, 1)
    x, y = _axis(nx, dx)[:, None, None], _axis(ny, dx)[None, :, None]
    r2 = x * x + y * y
    den = 1.0 + 2.0 * q * q * (tau * tau + r2) + q ** 4 * (tau * tau - r2) ** 2
    eps = C_SB * Tp ** 4 / q ** (4.0 / 3.0) * (2.0 * q) ** (8.0 / 3.0) / (tau * den) ** (4.0 / 3.0)
    a = 2.0 * q * q * tau / (1.0 + q * q * tau * tau + q * q * r2)
    vx, vy = a * x, a * y
    ut = 1.0 / torch.sqrt(1.0 - vx * vx - vy * vy)
    full = lambda t: t.expand(nx, ny, ne).contiguous()
    return dict(eps=full(eps), ux=full(ut * vx), uy=full(ut * vy),
                ue=torch.zeros(nx, ny, ne, dtype=F64, device=DEV))


def _tau0(c):
    return 1.0 if c["ic"] == "gubser" and not c["viscous"] else TAU0


def _event_ic(c, seed):
    if c["ic"] == "gubser":
        ic = _gubser(c["nx"], c["ny"], c["ne"], c["dx"], c["de"], _tau0(c), seed)
    else:
        ic = _hotspots(c["nx"], c["ny"], c["ne"], c["dx"], c["de"], seed)
    if c["bulk"]:
        ic["Pi"] = torch.zeros_like(ic["eps"])
        ic["nb"] = 0.3 * (ic["eps"] / ic["eps"].max()) ** 0.75
    return ic


def _desc(c, etas=ETAS):
    import paper_1802_04449_amd as K
    d = dict(nx=c["nx"], ny=c["ny"], ne=c["ne"], dx=c["dx"], dy=c["dx"], de=c["de"], h=c["h"],
             tau0=_tau0(c), viscous=int(c["viscous"]), etas=etas if c["viscous"] else 0.0,
             precision=K.KTMI_MIXED if c["precision"] == "mixed" else K.KTMI_FP64)
    if c["bulk"]:
        d.update(zetas=ZETAS, taubulk_coef=TAUBULK, baryon=1)
    return d


def _conformal(c):
    return c["ic"] == "gubser" and not c["viscous"]


def _batch_events(c):
    ev = []
    for s in c["events"].split(","):
        n, ne, etas = s.split("x")
        ev.append(dict(ic="hotspots", nx=int(n), ny=int(n), ne=int(ne), dx=0.16, de=0.3, h=0.01,
                       viscous=float(etas) > 0, etas=float(etas), precision=c["precision"],
                       bulk=False, steps=c["steps"]))
    return ev


def _capacity(c):
    return max(8192, c["nx"] * c["ny"] * c["ne"] // 16)


def _slices(c, seed):
    """Two slices 0.05 fm apart of an expanding, cooling hotspot event."""
    nx, ny, ne = c["nx"], c["ny"], c["ne"]
    eps = _hotspots(nx, ny, ne, c["dx"], c["de"], seed)["eps"]
    x = _axis(nx, c["dx"])[:, None, None]
    y = _axis(ny, c["dx"])[None, :, None]
    out = []
    for tau in (1.5, 1.55):
        e = eps * (TAU0 / tau) ** (4.0 / 3.0)
        v = 0.12 * tau
        ux, uy = v * x + 0.0 * e, v * y + 0.0 * e
        f = [e, ux, uy, 0.02 * torch.sin(x + y) + 0.0 * e]
        if c["with_pi"]:
            f += [e * (0.02 * math.cos(1.7 * m) / tau) * torch.cos(0.3 * m * x - 0.2 * y)
                  for m in range(10)]
        out.append(torch.stack(f).contiguous())
    return out[0], 1.5, out[1], 1.55


def _surface_records(n, seed):
    """Surface elements of the ranges that events give: (tau, x, y, eta), dSigma_mu, u~, pi~, e."""
    rng = np.random.default_rng(seed)
    r = np.zeros((n, 24))
    r[:, 0] = np.arange(n)
    r[:, 1] = rng.uniform(0.8, 9.0, n)
    rad, phi = 9.0 * np.sqrt(rng.random(n)), 2.0 * math.pi * rng.random(n)
    r[:, 2], r[:, 3] = rad * np.cos(phi), rad * np.sin(phi)
    r[:, 4] = rng.uniform(-4.5, 4.5, n)
    r[:, 5] = rng.gamma(1.0, 2e-3, n) * r[:, 1]
    r[:, 6:8] = rng.gamma(1.0, 2e-3, (n, 1)) * np.stack([np.cos(phi), np.sin(phi)], 1) * r[:, 1:2]
    r[:, 8] = 1e-3 * rng.standard_normal(n) * r[:, 1]
    v = 0.09 * rad + 0.05 * rng.standard_normal(n)
    r[:, 9], r[:, 10] = v * np.cos(phi), v * np.sin(phi)
    r[:, 11] = 0.05 * rng.standard_normal(n)
    r[:, 12:22] = 0.01 * rng.standard_normal((n, 10))
    r[:, 22] = 0.3
    return torch.as_tensor(r, device=DEV)


def _spectra_bins(c):
    mass = [0.13957, 0.13498, 0.49368, 0.49761, 0.93827, 0.93957, 1.11568, 1.18937, 0.77526,
            1.232, 1.01946, 1.67245]
    dof = [1.0, 1.0, 1.0, 1.0, 2.0, 2.0, 2.0, 2.0, 3.0, 4.0, 3.0, 4.0]
    stat = [-1, -1, -1, -1, 1, 1, 1, 1, -1, 1, -1, 0]
    ns = c["ns"]
    Y = np.linspace(-4.0, 4.0, c["nY"]) if c["nY"] > 1 else np.zeros(1)
    pt = 0.35 * np.polynomial.laguerre.laggauss(c["npt"])[0]
    phi = math.pi * (np.polynomial.legendre.leggauss(c["nphi"])[0] + 1.0)
    return (mass[:ns], dof[:ns], stat[:ns], [0.0] * ns), Y, pt, phi


T_FO, W_FO = 0.137, 0.4  # freeze-out temperature (GeV) and e + P (GeV/fm^3)


def _fluid_samples(n, seed):
    """(E, M, e) of random fluid states: e log-uniform, |v| uniform up to 0.99."""
    rng = np.random.default_rng(seed)
    e = np.exp(rng.uniform(math.log(1e-5), math.log(60.0), n))
    v = 0.99 * rng.random(n)
    t = _table()
    P = np.interp(e, t.deps * np.arange(len(t.P)), t.P)
    g2 = 1.0 / (1.0 - v * v)
    return (e + P) * g2 - P, (e + P) * g2 * v, e


def _network(seed):
    rng = np.random.default_rng(seed + 77)
    p = np.zeros(1249, dtype=np.float32)
    for a, b, lim in ((0, 128, 6.0 / 36), (160, 1184, 6.0 / 64), (1216, 1248, 6.0 / 33)):
        p[a:b] = rng.uniform(-math.sqrt(lim), math.sqrt(lim), b - a)
    return p


LR = 3e-3


# ---------------------------------------------------------------------------
# Preparation and one pass
# ---------------------------------------------------------------------------

def prepare(case, seed):
    import paper_1802_04449_amd as K
    c = case
    if c["kind"] == "evolve":
        h = K.Hydro(device=DEV, **_desc(c))
        h.set_eos("conformal" if _conformal(c) else _table())
        return dict(c=c, h=h, ic=_event_ic(c, seed))
    if c["kind"] == "batch":
        st = torch.cuda.Stream()
        hs, ics = [], []
        for k, e in enumerate(_batch_events(c)):
            h = K.Hydro(device=DEV, stream=st, **_desc(e, e["etas"]))
            h.set_eos(_table())
            ics.append(_event_ic(e, seed + 1000 * k))
            hs.append(h)
        torch.cuda.synchronize()
        for h, ic in zip(hs, ics):
            h.set_initial(ic)
        g = K.Group(hs)
        g.set_graph(True)
        return dict(c=c, hs=hs, g=g, ics=ics, st=st)
    if c["kind"] == "surface":
        h = K.Hydro(device=DEV, nx=c["nx"], ny=c["ny"], ne=c["ne"], dx=c["dx"], dy=c["dx"],
                    de=c["de"], h=0.01, tau0=TAU0, viscous=1, etas=ETAS)
        h.set_eos(_table())
        # the program's record buffer, kept from one pair of slices to the next
        out = torch.zeros(_capacity(c), K.KTMI_SURF_REC, dtype=F64, device=DEV)
        return dict(c=c, h=h, s=_slices(c, seed), out=out,
                    count=torch.zeros(1, dtype=torch.int64, device=DEV))
    if c["kind"] == "spectra":
        return dict(c=c, el=_surface_records(c["n"], seed), bins=_spectra_bins(c))
    from paper_1802_04449_amd import mlp
    tr = mlp.Trainer(*_fluid_samples(c["batch"], seed), device=DEV,
                     mode=K.KTMI_MLP_BF16 if c["mode"] == "bf16" else K.KTMI_MLP_FP32)
    tr.params.copy_(torch.as_tensor(_network(seed)))
    return dict(c=c, tr=tr)


def _fields(s):
    """A slice (e, u~[, pi~]) by its fields, whole."""
    return dict(e=s[0], u=s[1:4], pi=s[4:]) if s.shape[0] > 4 else dict(e=s[0], u=s[1:4])


def _record_fields(r):
    """Surface records by their fields, whole: hypercube, centre, dSigma, u~, pi~, e (and zero)."""
    return dict(cube=r[:, 0], centre=r[:, 1:5], normal=r[:, 5:9], u=r[:, 9:12], pi=r[:, 12:22],
                e=r[:, 22:])


def run(state):
    c = state["c"]
    if c["kind"] == "evolve":
        h = state["h"]
        h.set_initial(state["ic"])
        if c["check"]:
            h.step_until(1e-3, c["steps"], c["check"])
        else:
            h.step(c["steps"])
        out = _fields(h.snapshot(c["viscous"]))
        out["T"] = [h.read("T%d" % m) for m in range(4)]
        if c["bulk"]:
            out["Pi"], out["nb"] = h.read("Pi"), h.read("nb")
        d = h.diag()
        out["diag"] = dict(eps_max=d["eps_max"], sum_Ttt=d["sum_Ttt"], tau=d["tau"])
        return out
    if c["kind"] == "batch":
        with torch.cuda.stream(state["st"]):
            for h, ic in zip(state["hs"], state["ics"]):
                h.set_initial(ic)
            state["g"].step(c["steps"])
            return [_fields(h.snapshot(bool(h.desc.viscous))) for h in state["hs"]]
    if c["kind"] == "surface":
        import paper_1802_04449_amd as K
        A, ta, B, tb = state["s"]
        K.ktmi_surface(state["h"].h, A.data_ptr(), ta, B.data_ptr(), tb, c["with_pi"], c["eps_f"],
                       state["out"].data_ptr(), _capacity(c), state["count"].data_ptr())
        return dict(count=state["count"], **_record_fields(state["out"]))
    if c["kind"] == "spectra":
        import paper_1802_04449_amd as K
        species, Y, pt, phi = state["bins"]
        return K.spectra(state["el"], T_FO, W_FO if c["df"] else 0.0, species, Y, pt, phi)
    tr = state["tr"]
    tr.step(c["batch"], lr=LR)
    return dict(params=tr.params, m=tr.m, v=tr.v, grad=tr.out[:1249], loss=tr.out[1249:1250],
                count=tr.out[1250:])


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------

def _evolve_work(c):
    """State read once and written once per step (u~ of two times, pi~, T~, e) plus the result
    written and read out; operations of the cells with matter only (a disk of about 9 fm and the
    eta plateau for hotspots): per step two flux evaluations on three axes (about 450 operations
    per cell and axis, 180 without pi~), two sources (400 / 20) and two root solves (150)."""
    n = c["nx"] * c["ny"] * c["ne"]
    nq = (12 if c["bulk"] else 10) if c["viscous"] else 0
    qb = 4 if c["precision"] == "mixed" else 8
    hot = 1.0
    if c["ic"] == "hotspots":
        hot = min(1.0, math.pi * 9.0 ** 2 / (c["nx"] * c["ny"] * c["dx"] ** 2))
        hot *= min(1.0, 12.0 / (c["ne"] * c["de"])) if c["ne"] > 1 else 1.0
    axes = 3 if c["ne"] > 1 else 2
    ops = 2 * axes * (450 if nq else 180) + 2 * (400 if nq else 20) + 300
    per = 2 * (11 * 8 + nq * qb)
    return dict(bytes=n * (per * c["steps"] + (4 + 8 + nq) * 8), flops=n * hot * ops * c["steps"])


def work(case):
    c = case
    if c["kind"] == "evolve":
        return _evolve_work(c)
    if c["kind"] == "batch":
        w = [_evolve_work(e) for e in _batch_events(c)]
        return dict(bytes=sum(x["bytes"] for x in w), flops=sum(x["flops"] for x in w))
    if c["kind"] == "surface":
        # e of both slices; a record and the other fields of a corner cell for the elements,
        # about a hundredth of the cells
        n = c["nx"] * c["ny"] * c["ne"]
        nf = 14 if c["with_pi"] else 4
        return dict(bytes=16 * n + n // 100 * (192 + 16 * (nf - 1)), flops=n // 100 * 2000.0)
    if c["kind"] == "spectra":
        # per element and bin: 22 operations with delta f, 14 without (the exponential's factors
        # and the longitudinal terms are shared by many bins)
        bins = c["ns"] * c["nY"] * c["npt"] * c["nphi"]
        return dict(bytes=192 * c["n"] + 8 * bins, flops=(22.0 if c["df"] else 14.0) * c["n"] * bins)
    # forward, backward to the hidden layer and both weight gradients: three products of 32 x 32
    # and three of 4 x 32 per sample; the samples once, the parameters and moments once
    n = c["batch"]
    return dict(bytes=24 * n + 8 * 1249 * 4, flops=n * 2.0 * (3 * 1024 + 2 * 128 + 3 * 32))


# ---------------------------------------------------------------------------
# The same results in plain torch FP64
# ---------------------------------------------------------------------------

SYM = [[0, 1, 2, 3], [1, 4, 5, 6], [2, 5, 7, 8], [3, 6, 8, 9]]


class _Eos:
    def __init__(self, conformal):
        self.t = None
        if not conformal:
            t = _table()
            self.t = [torch.as_tensor(a, device=DEV) for a in (t.P, t.T, t.cs2)]
            self.inv, self.n = 1.0 / t.deps, len(t.P)

    def __call__(self, e):
        """P, T, cs2 and dP/de; past the last row P keeps its slope, cs2 is held and
        T = T_last ((e + P)/(e + P)_last)^(1/4)."""
        e = e.clamp(min=0.0)
        if self.t is None:
            third = torch.full_like(e, 1.0 / 3.0)
            return e / 3.0, (e / C_SB) ** 0.25, third, third
        x = e * self.inv
        i = x.floor().long().clamp(max=self.n - 2)
        f = x - i
        P, T, c = self.t
        d = P[i + 1] - P[i]
        Pe, fc = P[i] + f * d, f.clamp(max=1.0)
        last = (self.n - 1) / self.inv + P[-1]
        Te = torch.where(f > 1.0, T[-1] * ((e + Pe) / last) ** 0.25,
                         T[i] + fc * (T[i + 1] - T[i]))
        return Pe, Te, c[i] + fc * (c[i + 1] - c[i]), d * self.inv


def _ut(u):
    return torch.sqrt(1.0 + u[0] ** 2 + u[1] ** 2 + u[2] ** 2)


def _flux_div(eos, e, u, pi, Pi, nb, deltas, tau, with_T, with_pi):
    """-(H_{+1/2} - H_{-1/2})/Delta summed over the axes, of T~ (4) and of pi~ (, Pi, n)."""
    q = [e] + list(u) + (list(pi) if pi is not None else [])
    if Pi is not None:
        q += [Pi, nb]
    nq = len(q) - 4
    RT = [torch.zeros_like(e) for _ in range(4)] if with_T else None
    Rq = [torch.zeros_like(e) for _ in range(nq)] if with_pi else None
    for d in range(3):
        n = e.shape[d]
        if n == 1:
            continue
        idx = torch.arange(-2, n + 2, device=DEV).clamp(0, n - 1)
        L, R = [], []
        for v in q:
            p = v.index_select(d, idx)
            a, b, c_, f = (p.narrow(d, t, n + 1) for t in range(4))

            def slope(m, z, r):
                s = torch.stack([THETA * (z - m), 0.5 * (r - m), THETA * (r - z)])
                return s.amin(0).clamp(min=0.0) + s.amax(0).clamp(max=0.0)
            L.append(b + 0.5 * slope(a, b, c_))
            R.append(c_ - 0.5 * slope(b, c_, f))
        side = []
        for s in (L, R):
            ut = _ut(s[1:4])
            P, _, cs2, _ = eos(s[0])
            if Pi is not None:
                P = P + s[4 + nq - 2]
            w = s[0].clamp(min=0.0) + P
            ud = s[1 + d]
            u2 = s[1] ** 2 + s[2] ** 2 + s[3] ** 2
            z = 1.0 - cs2
            disc = 1.0 + (u2 - ud * ud).clamp(min=0.0) * z
            speed = (ud.abs() * z * ut + torch.sqrt(cs2 * disc)) / (1.0 + u2 * z)
            side.append((s, ut, P, w, ud, speed))
        c = torch.maximum(side[0][5], side[1][5])
        delta = deltas[d] * (tau if d == 2 else 1.0)

        def add(R_, Q, F):
            H = 0.5 * (F[0] + F[1]) - 0.5 * c * (Q[1] - Q[0])
            R_ -= (H.narrow(d, 1, n) - H.narrow(d, 0, n)) / delta
        if with_T:
            for nu in range(4):
                Q, F = [], []
                for s, ut, P, w, ud, _ in side:
                    un = ut if nu == 0 else s[nu]
                    p0 = s[4 + SYM[0][nu]] if pi is not None else 0.0
                    pd = s[4 + SYM[d + 1][nu]] if pi is not None else 0.0
                    Q.append(tau * (w * ut * un - (P if nu == 0 else 0.0) + p0))
                    F.append(tau * (w * ud * un + (P if nu == d + 1 else 0.0) + pd))
                add(RT[nu], Q, F)
        if with_pi:
            for m in range(nq):
                add(Rq[m], [t[1] * t[0][4 + m] for t in side], [t[4] * t[0][4 + m] for t in side])
        del L, R, side
    return RT, Rq


def _root(eos, K, Pi):
    """(e, u~) of K = T~/tau - pi~; zero below the cutoff."""
    E = K[0]
    B = E if Pi is None else E + Pi.clamp(max=0.0)
    out = [torch.zeros_like(E) for _ in range(4)]
    act = (E >= EPS_CUT) & (B > 0.0)
    E, B = E[act], B[act]
    k = [x[act] for x in K[1:]]
    Pb = torch.zeros_like(E) if Pi is None else Pi[act]
    M2 = k[0] ** 2 + k[1] ** 2 + k[2] ** 2
    cap = (1.0 - 1e-10) * B
    s = torch.where(M2 > cap * cap, cap / torch.sqrt(M2), torch.ones_like(M2))
    k = [x * s for x in k]
    M2 = k[0] ** 2 + k[1] ** 2 + k[2] ** 2
    lo0 = (E - M2 / B).clamp(min=0.0)
    lo, hi, x = lo0.clone(), E.clone(), E.clone()
    if E.numel():
        for _ in range(200):
            P, _, _, dP = eos(x)
            r = 1.0 / (E + P + Pb)
            f = x - E + M2 * r
            hi, lo = torch.where(f > 0, x, hi), torch.where(f > 0, lo, x)
            xn = x - f / (1.0 - M2 * dP * r * r)
            xn = torch.where((xn >= lo) & (xn <= hi), xn, 0.5 * (lo + hi))
            far = ((xn - x).abs() > 2e-15 * xn).any()
            x = xn
            if not bool(far):
                break
    P = eos(x)[0] + Pb
    inv = 1.0 / torch.sqrt((E + P) * (x + P))
    keep = x >= EPS_CUT
    for o, v in zip(out, [x] + [t * inv for t in k]):
        o[act] = torch.where(keep, v, torch.zeros_like(v))
    return out[0], out[1:]


def _pi_source(eos, e, u, uE, uL, pi, Pi, nb, deltas, tau, h, etas):
    uc = [_ut(u)] + list(u)
    G = [[(b - a) / h for a, b in zip([_ut(uE)] + list(uE), [_ut(uL)] + list(uL))]]
    for d in range(3):
        n = e.shape[d]
        ip = (torch.arange(n, device=DEV) + 1).clamp(max=n - 1)
        im = (torch.arange(n, device=DEV) - 1).clamp(min=0)
        half = 0.5 / (deltas[d] * (tau if d == 2 else 1.0))
        G.append([(v.index_select(d, ip) - v.index_select(d, im)) * half for v in uc])
    G[3][0] = G[3][0] + uc[3] / tau
    G[3][3] = G[3][3] + uc[0] / tau
    theta = G[0][0] + G[1][1] + G[2][2] + G[3][3]
    a = [sum(uc[m] * G[m][nu] for m in range(4)) for nu in range(4)]
    g = [1.0, -1.0, -1.0, -1.0]
    b = [sum(g[m] * pi[SYM[nu][m]] * a[m] for m in range(4)) for nu in range(4)]
    P, T, _, _ = eos(e)
    rate = T / (TAUPI * etas * HBARC)
    ue, S = uc[3], []
    inhom = {0: lambda: 2.0 * pi[3], 9: lambda: 2.0 * pi[3], 1: lambda: pi[6], 2: lambda: pi[8],
             3: lambda: pi[0] + pi[9], 6: lambda: pi[1], 8: lambda: pi[2]}
    for mu in range(4):
        for nu in range(mu, 4):
            m = SYM[mu][nu]
            proj = (g[mu] if mu == nu else 0.0) - uc[mu] * uc[nu]
            sig = (g[mu] * G[mu][nu] + g[nu] * G[nu][mu] - uc[mu] * a[nu] - uc[nu] * a[mu]
                   - 2.0 / 3.0 * proj * theta)
            s = (-pi[m] * rate + (e + P) / TAUPI * sig - pi[m] * theta / 3.0
                 - (uc[mu] * b[nu] + uc[nu] * b[mu]))
            I = ue * inhom[m]() if m in inhom else 0.0
            S.append(s - (pi[m] * uc[0] + I) / tau)
    if Pi is not None:
        S.append(-Pi * T / (TAUBULK * ZETAS * HBARC) - (e + P) / TAUBULK * theta - Pi * theta / 3.0
                 - Pi * uc[0] / tau)
        S.append(-nb * uc[0] / tau)
    on = e >= EPS_CUT
    return [torch.where(on, s, torch.zeros_like(s)) for s in S]


def _regulate(eos, e, q):
    """pi~ scaled to sqrt|pi:pi| <= 0.3 (e + P), Pi clipped to [-P, P], all zero where e = 0."""
    P = eos(e)[0]
    w = e + P
    p = q[:10]
    pp = (p[0] ** 2 + p[4] ** 2 + p[7] ** 2 + p[9] ** 2 - 2.0 * (p[1] ** 2 + p[2] ** 2 + p[3] ** 2)
          + 2.0 * (p[5] ** 2 + p[6] ** 2 + p[8] ** 2))
    rho = torch.sqrt(pp.abs()) / torch.where(w > 0, w, torch.ones_like(w))
    f = torch.where(rho > PI_REG, PI_REG / rho, torch.ones_like(rho))
    out = [x * f for x in p]
    if len(q) > 10:
        out += [torch.minimum(torch.maximum(q[10], -P), P), q[11]]
    return [torch.where(w > 0, x, torch.zeros_like(x)) for x in out]


def _exact_event(c, seed, etas):
    eos = _Eos(_conformal(c))
    ic = _event_ic(c, seed)
    deltas, h, tau, visc = (c["dx"], c["dx"], c["de"]), c["h"], _tau0(c), c["viscous"]
    e = torch.where(ic["eps"] >= EPS_CUT, ic["eps"], torch.zeros_like(ic["eps"]))
    on = e > 0
    u = [torch.where(on, ic[k], torch.zeros_like(e)) for k in ("ux", "uy", "ue")]
    nq = (12 if c["bulk"] else 10) if visc else 0
    q = [torch.zeros_like(e) for _ in range(nq)]
    if c["bulk"]:
        q[10], q[11] = torch.where(on, ic["Pi"], q[10]), torch.where(on, ic["nb"], q[11])
    del ic

    def split(q):
        return (q[:10] if visc else None), (q[10] if nq == 12 else None), (q[11] if nq == 12 else None)

    def geometric(R, e, u, q):
        P = eos(e)[0]
        if nq == 12:
            P = P + q[10]
        w, ut = e + P, _ut(u)
        R[0] = R[0] - (w * u[2] ** 2 + P + (q[9] if visc else 0.0))
        R[3] = R[3] - (w * ut * u[2] + (q[3] if visc else 0.0))

    P, ut = eos(e)[0], _ut(u)
    if nq == 12:
        P = P + q[10]
    T = [tau * ((e + P) * ut * x - (P if k == 0 else 0.0)) for k, x in enumerate([ut] + u)]
    # one ideal forward-Euler step gives u~ at the time before the first
    Pe = eos(e)[0]
    R, _ = _flux_div(eos, e, u, None, None, None, deltas, tau, True, False)
    R[0] = R[0] - ((e + Pe) * u[2] ** 2 + Pe)
    R[3] = R[3] - (e + Pe) * ut * u[2]
    K = [(tau * ((e + Pe) * ut * x - (Pe if k == 0 else 0.0)) + h * R[k]) / (tau + h)
         for k, x in enumerate([ut] + u)]
    up = [2.0 * a - b for a, b in zip(u, _root(eos, K, None)[1])]
    for _ in range(c["steps"]):
        tau1 = tau + h
        pi, Pi, nb = split(q)
        R, Rq = _flux_div(eos, e, u, pi, Pi, nb, deltas, tau, True, visc)
        geometric(R, e, u, q)
        utn, us = _ut(u), _ut([2.0 * a - b for a, b in zip(u, up)])
        q1 = []
        if visc:
            S = _pi_source(eos, e, u, up, u, pi, Pi, nb, deltas, tau, h, etas)
            q1 = _regulate(eos, e, [(utn * x + h * (r + s)) / us for x, r, s in zip(q, Rq, S)])
        T1 = [t + h * r for t, r in zip(T, R)]
        K = [t / tau1 - (q1[k] if visc else 0.0) for k, t in enumerate(T1)]
        e1, u1 = _root(eos, K, q1[10] if nq == 12 else None)
        qn = []
        if visc:
            pi1, Pi1, nb1 = split(q1)
            _, Rq = _flux_div(eos, e1, u1, pi1, Pi1, nb1, deltas, tau1, False, True)
            S = _pi_source(eos, e1, u1, u, u1, pi1, Pi1, nb1, deltas, tau1, h, etas)
            ut1 = _ut(u1)
            qn = _regulate(eos, e1, [(0.5 * (utn * a + us * b) + 0.5 * h * (r + s)) / ut1
                                     for a, b, r, s in zip(q, q1, Rq, S)])
        pin, Pin, nbn = split(qn)
        R, _ = _flux_div(eos, e1, u1, pin, Pin, nbn, deltas, tau1, True, False)
        geometric(R, e1, u1, qn)
        T = [t + 0.5 * ((t1 - t) + h * r) for t, t1, r in zip(T, T1, R)]
        K = [t / tau1 - (qn[k] if visc else 0.0) for k, t in enumerate(T)]
        up = u
        e, u = _root(eos, K, qn[10] if nq == 12 else None)
        q = [torch.where(e > 0, x, torch.zeros_like(x)) for x in qn]
        tau = tau1
    return e, u, q, T, tau


def _exact_surface(c, seed):
    A, ta, B, tb = _slices(c, seed)
    n3 = (c["nx"], c["ny"], c["ne"])
    ext = (tb - ta, c["dx"], c["dx"], c["de"])
    nc = [max(n - 1, 1) for n in n3]
    corner = list(itertools.product((0, 1), repeat=4))

    def at(v, bits):  # v of slice A or B at the corner, for every hypercube
        s = (A, B)[bits[0]][v]
        for d in range(3):
            s = s.narrow(d, bits[1 + d] if n3[d] > 1 else 0, nc[d])
        return s
    hot = sum(((at(0, b) - c["eps_f"]) > 0).int() for b in corner)
    ids = torch.nonzero(((hot > 0) & (hot < 16)).reshape(-1)).reshape(-1)
    phi = {b: at(0, b).reshape(-1)[ids] - c["eps_f"] for b in corner}

    def tet(v):
        """Hot fraction of a tetrahedron from its sorted vertex values."""
        v = torch.stack(v).sort(0).values
        k = (v > 0).sum(0)
        one = torch.ones_like(v[0])

        def ratio(a, b):
            d = a - b
            return torch.where(d != 0, a / torch.where(d != 0, d, one), one)
        f1 = ratio(v[3], v[0]) * ratio(v[3], v[1]) * ratio(v[3], v[2])
        f3 = 1.0 - ratio(v[0], v[3]) * ratio(v[0], v[2]) * ratio(v[0], v[1])
        a, b, m, d = v[2], v[3], -v[0], -v[1]
        f2 = ((a * a * b * b + a * b * (a + b) * (m + d) + m * d * (a * a + a * b + b * b))
              / torch.where(k == 2, (a + m) * (a + d) * (b + m) * (b + d), one))
        z = torch.zeros_like(one)
        return torch.where(k == 1, f1, torch.where(k == 2, f2, torch.where(k == 3, f3, torch.where(
            k == 4, one, z))))

    def cube(w):
        s = 0.0
        for order in itertools.permutations(range(3)):
            p, path = [0, 0, 0], []
            for ax in (None,) + order:
                if ax is not None:
                    p[ax] = 1
                path.append(w[tuple(p)])
            s = s + tet(path)
        return s / 6.0
    S = []
    for mu in range(4):
        f = [cube({b[:mu] + b[mu + 1:]: phi[b] for b in corner if b[mu] == s}) for s in (0, 1)]
        V = math.prod(ext[a] for a in range(4) if a != mu)
        S.append(V * (f[0] - f[1]))
    cen, cnt = [torch.zeros_like(phi[corner[0]]) for _ in range(4)], 0.0
    for b in corner:
        for ax in range(4):
            if b[ax]:
                continue
            b2 = b[:ax] + (1,) + b[ax + 1:]
            x = ((phi[b] > 0) != (phi[b2] > 0)).double()
            d = phi[b] - phi[b2]
            s = phi[b] / torch.where(d != 0, d, torch.ones_like(d))
            for a in range(4):
                cen[a] = cen[a] + x * (s if a == ax else float(b[a]))
            cnt = cnt + x
    cen = [x / cnt for x in cen]
    out = torch.zeros(ids.numel(), 24, dtype=F64, device=DEV)
    out[:, 0] = ids.double()
    out[:, 1] = ta + cen[0] * ext[0]
    ijk = [t.double() for t in (ids // (nc[1] * nc[2]), ids // nc[2] % nc[1], ids % nc[2])]
    for d in range(3):
        out[:, 2 + d] = ((ijk[d] - 0.5 * (n3[d] - 1)) * ext[1 + d]
                         + (cen[1 + d] * ext[1 + d] if n3[d] > 1 else 0.0))
    for mu in range(4):
        out[:, 5 + mu] = out[:, 1] * S[mu]
    for v in range(A.shape[0]):
        s = 0.0
        for b in corner:
            w = math.prod((cen[a] if b[a] else 1.0 - cen[a]) for a in range(4))
            s = s + w * at(v, b).reshape(-1)[ids]
        out[:, 22 if v == 0 else 8 + v] = s
    return out


def _exact_spectra(c, seed):
    el = _surface_records(c["n"], seed)
    (mass, dof, stat, mu), Y, pt, phi = _spectra_bins(c)
    ct = lambda a: torch.as_tensor(np.asarray(a, dtype=np.float64), device=DEV)
    px = (ct(pt)[:, None] * torch.cos(ct(phi))[None, :]).reshape(-1)
    py = (ct(pt)[:, None] * torch.sin(ct(phi))[None, :]).reshape(-1)
    ptb = ct(pt)[:, None].expand(-1, c["nphi"]).reshape(-1)
    out = torch.zeros(c["ns"], c["nY"], c["npt"], c["nphi"], dtype=F64, device=DEV)
    pref = 1.0 / (2.0 * math.pi * HBARC) ** 3
    tau, eta = el[:, 1:2], el[:, 4:5]
    dS, u, p = el[:, 5:9], el[:, 9:12], el[:, 12:22]
    ut = torch.sqrt(1.0 + (u * u).sum(1, keepdim=True))
    chunk = max(1, int(3e7) // px.numel())
    for s in range(c["ns"]):
        mT = torch.sqrt(mass[s] ** 2 + ptb * ptb)[None, :]
        for iy in range(c["nY"]):
            acc = torch.zeros_like(px)
            for a in range(0, c["n"], chunk):
                z = slice(a, a + chunk)
                yr = float(Y[iy]) - eta[z]
                p0, p3 = mT * torch.cosh(yr), mT * torch.sinh(yr)
                pds = p0 * dS[z, 0:1] + px * dS[z, 1:2] + py * dS[z, 2:3] + p3 / tau[z] * dS[z, 3:4]
                pu = p0 * ut[z] - px * u[z, 0:1] - py * u[z, 1:2] - p3 * u[z, 2:3]
                f = 1.0 / (torch.exp((pu - mu[s]) / T_FO) + stat[s])
                if c["df"]:
                    q = (p0, -px, -py, -p3)
                    pp = sum((1.0 if i == j else 2.0) * q[i] * q[j] * p[z, SYM[i][j]:SYM[i][j] + 1]
                             for i in range(4) for j in range(i, 4))
                    f = f * (1.0 + (1.0 - stat[s] * f) * pp / (2.0 * T_FO * T_FO * W_FO))
                acc += (pds * f).sum(0)
            out[s, iy] = (dof[s] * pref * acc).reshape(c["npt"], c["nphi"])
    return out


def _exact_train(c, seed):
    E, M, e = (torch.as_tensor(a, device=DEV) for a in _fluid_samples(c["batch"], seed))
    p = torch.as_tensor(_network(seed).astype(np.float64), device=DEV).requires_grad_()
    lo = (E - M * M / E).clamp(min=0.0)
    r = M / E
    f = torch.stack([0.2 * torch.log(E), r, r * r, 0.1 * torch.log((lo / E).clamp(min=1e-30))], 1)
    h1 = torch.tanh(f @ p[:128].view(32, 4).T + p[128:160])
    h2 = torch.tanh(h1 @ p[160:1184].view(32, 32).T + p[1184:1216])
    guess = lo + torch.sigmoid(h2 @ p[1216:1248] + p[1248]) * (E - lo)
    loss = (((guess - e) / E) ** 2).mean()
    g, = torch.autograd.grad(loss, p)
    p, g, loss = p.detach(), g.detach(), loss.detach()
    # first Adam step with zero moments (bias corrections cancel the decays)
    return dict(params=p - LR * g / (g.abs() + 1e-8), m=0.1 * g, v=0.001 * g * g, grad=g,
                loss=loss.view(1), count=torch.tensor([float(c["batch"])], dtype=F64, device=DEV))


def exact(case, seed):
    c = case
    if c["kind"] == "evolve":
        e, u, q, T, tau = _exact_event(c, seed, ETAS)
        out = dict(T=T, **_fields(torch.stack([e] + list(u) + q[:10])))
        if c["bulk"]:
            out["Pi"], out["nb"] = q[10], q[11]
        out["diag"] = dict(eps_max=float(e.max()), tau=tau,
                           sum_Ttt=float(T[0].sum()) * c["dx"] ** 2 * c["de"])
        return out
    if c["kind"] == "batch":
        out = []
        for k, ev in enumerate(_batch_events(c)):
            e, u, q, _, _ = _exact_event(ev, seed + 1000 * k, ev["etas"])
            out.append(_fields(torch.stack([e] + list(u) + q)))
        return out
    if c["kind"] == "surface":
        el, cap = _exact_surface(c, seed), _capacity(c)
        rec = torch.zeros(cap, 24, dtype=F64, device=DEV)
        rec[:min(cap, len(el))] = el[:cap]
        return dict(count=torch.tensor([len(el)], device=DEV), **_record_fields(rec))
    if c["kind"] == "spectra":
        return _exact_spectra(c, seed)
    return _exact_train(c, seed)
