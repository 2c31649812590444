"""The spectra kernel over the shapes its launch rule tells apart (few or many
(species, Y) pairs, one or many phi bins, bins that do not fill a tile, slices that
do not fill a stage) against the CPU oracle, and its factored exponential where one
factor alone leaves the FP64 range.

Both sides evaluate the same formula in FP64; the bar is that of the other spectra
tests, 1e-12 of the species' largest bin plus 1e-11 of the bin itself: the exponent
(p.u - mu)/T is a difference of terms up to ~2e3 here, each rounded to 2^-53 of
itself, so f carries up to ~1e-12 relative."""
import math
import sys

import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

MASS = [0.13957, 0.49368, 0.93827, 1.232, 0.77526]
DOF = [1.0, 1.0, 2.0, 4.0, 3.0]
STAT = [-1, 0, 1, 1, -1]
MU = [0.05, 0.0, 0.2, -0.1, 0.0]


def _records(n, seed, umax=1.2):
    rng = np.random.default_rng(seed)
    r = np.zeros((n, 24))
    r[:, 1] = rng.uniform(0.6, 10.0, n)
    r[:, 4] = rng.uniform(-5.0, 5.0, n)
    r[:, 5:9] = 1e-2 * rng.standard_normal((n, 4)) * r[:, 1:2]
    r[:, 9:12] = umax * rng.uniform(-1.0, 1.0, (n, 3)) * np.array([1.0, 1.0, 0.2])
    r[:, 12:22] = 0.02 * rng.standard_normal((n, 10))
    return r


def _check(r, T, wP, ns, Y, pt, phi, label):
    import torch

    import paper_1802_04449_amd as K
    print(f"[gpu-case] spectra {label}", flush=True)
    sys.stdout.flush()
    sp = (MASS[:ns], DOF[:ns], STAT[:ns], MU[:ns])
    g = K.spectra(torch.as_tensor(r).cuda(), T, wP, sp, Y, pt, phi).cpu().numpy()
    o = O.spectra(r, T, wP, sp, Y, pt, phi)
    assert np.abs(o).max() > 0 and np.all(np.isfinite(g))
    scale = np.abs(o).reshape(ns, -1).max(axis=1)[:, None, None, None]
    bad = np.abs(g - o) > 1e-12 * scale + 1e-11 * np.abs(o)
    assert not bad.any(), (label, float((np.abs(g - o) / scale).max()), np.argwhere(bad)[:5].tolist())


@pytest.mark.parametrize("delta_f", [False, True])
@pytest.mark.parametrize("ns,nY,npt,nphi", [(1, 1, 1, 1), (1, 17, 2, 9), (3, 23, 2, 48), (5, 13, 3, 1),
                                            (1, 16, 17, 1), (5, 26, 1, 4), (2, 33, 5, 5),
                                            (1, 3, 2, 17)])
def test_shapes(ns, nY, npt, nphi, delta_f):
    Y = np.linspace(-2.0, 2.0, nY) if nY > 1 else np.array([0.3])
    pt = np.linspace(0.05, 3.0, npt)
    phi = np.linspace(0.1, 2.0 * math.pi, nphi)
    for n, seed in ((1, 3), (519, 4)):
        _check(_records(n, seed), 0.137, 0.4 if delta_f else 0.0, ns, Y, pt, phi,
               f"{ns}x{nY}x{npt}x{nphi} n={n} delta_f={delta_f}")


def test_exponent_range():
    """pT u / T up to 1300 with p.u / T of a few hundred, and rapidity distances whose
    exponent alone overflows."""
    r = _records(301, 8, umax=3.0)
    r[:, 11] = 0.0
    r[::7, 4] += 20.0
    _check(r, 0.137, 0.0, 3, np.array([-1.0, 0.0, 6.0]), np.array([0.5, 20.0, 60.0]),
           np.linspace(0.0, 2.0 * math.pi, 13), "exponent range")


def test_smallest_workspace():
    """A workspace for the fewest slices (256 elements each) gives the same spectra as one
    of the size asked for, up to the order of the sums; less than that is refused."""
    import torch

    import paper_1802_04449_amd as K
    n, ns, nY, npt, nphi = 519, 2, 3, 4, 7
    r = torch.as_tensor(_records(n, 5)).cuda()
    Y, pt, phi = np.linspace(-1, 1, nY), np.linspace(0.1, 2, npt), np.linspace(0, 6, nphi)
    nbins = ns * nY * npt * nphi
    tables = (4 * ns + nY + npt + 2 * nphi + 31) // 32 * 32
    need, asked = 8 * (tables + 3 * nbins), K.ktmi_spectra_workspace_bytes(n, ns, nY, npt, nphi)
    assert asked > need
    ws = torch.empty(asked // 8, dtype=torch.float64, device="cuda")
    got = []
    for nb in (asked, need):
        out = torch.full((nbins,), float("nan"), dtype=torch.float64, device="cuda")
        K.ktmi_spectra(r.data_ptr(), n, 0.15, 0.4, MASS[:ns], DOF[:ns], STAT[:ns], MU[:ns], Y, pt,
                       phi, out.data_ptr(), ws.data_ptr(), nb, 0)
        torch.cuda.synchronize()
        got.append(out.cpu().numpy())
    # n terms added in another order: n 2^-53 of the sum of their magnitudes
    np.testing.assert_allclose(got[0], got[1], rtol=0, atol=n * 2.0 ** -53 * np.abs(got[0]).max() * 10)
    with pytest.raises(K.KtmiError):
        K.ktmi_spectra(r.data_ptr(), n, 0.15, 0.4, MASS[:ns], DOF[:ns], STAT[:ns], MU[:ns], Y, pt,
                       phi, out.data_ptr(), ws.data_ptr(), need - 8, 0)
