"""The gradient kernel where its work splits: part of a wave's 64 samples, one wave,
one workgroup (4 waves) and one sample more, and more samples than the largest grid
takes in one sweep (512 workgroups x 256), some of them below emin.  Against the FP64
reference network; the bars are those of the other gradient tests (FP32 forward and
backward: 1e-5 of max |g|, BF16 forward 2e-2)."""
import numpy as np
import pytest

import oracle as O
from tests.test_zz_no_alloc import _run, _samples

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,tol", [(0, 1e-5), (1, 2e-2)])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 255, 256, 257, 131072, 131137])
def test_gradient_at_chunk_edges(n, mode, tol):
    print(f"gradient: mode={mode} n={n}", flush=True)
    p32 = np.random.default_rng(3).normal(0.0, 0.4, 1249).astype(np.float32)
    E, M, eps = _samples(n, 31 + n)
    emin = 1e-7
    if n > 2:
        E[n // 2] = M[n // 2] = 0.0  # below emin: left out
        emin = float(np.partition(E, n // 5)[n // 5])
    keep = E >= emin
    L, ref = O.mlp_loss_grad(p32.astype(np.float64), E[keep], M[keep], eps[keep])
    for which in ("ws", "noalloc"):
        out = _run(which, p32, E, M, eps, mode, emin=emin)
        assert out[-1] == keep.sum()
        assert np.abs(out[:1249] - ref).max() <= tol * np.abs(ref).max()
        assert out[-2] == pytest.approx(L, rel=tol)
