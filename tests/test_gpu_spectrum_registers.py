"""The spectrum's register transforms (64, 128 and 256 nodes a side) against NumPy's FFT, at
ensembles that fill a block's sixteen lines, leave some empty or need several blocks, and
next to a size that takes the general passes.

Tolerance: 1e-10 relative per shell, as for the general passes (sums of n^2 M positive terms
and transforms of at most 256 points in FP64).
"""
import numpy as np
import pytest

from paper_2308_03972_amd import binding
from gpu_helpers import cuda, host, need_gpu, random_state, say

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("n,M,storage", [(64, 1, 0), (64, 17, 0), (64, 16, 1), (128, 5, 0),
                                         (128, 33, 1), (256, 3, 0), (256, 18, 1), (96, 5, 0)])
def test_register_transforms_match_fft(n, M, storage):
    say(f"spectrum in registers: {n}^2 x {M}, storage {storage}")
    rng = np.random.default_rng(600 + n + M)
    fe = random_state(rng, M, n, n)
    ctx = binding.Context(n, n, M, 0.55, 0.1, np.array([[1, 1]], np.int32), 2, (0.1, 0.1), 4.0, 1.05,
                          storage=(binding.STORAGE_F64, binding.STORAGE_F32_DEV)[storage])
    f = ctx.import_canonical(cuda(fe))
    fe = host(ctx.export_canonical(f))
    kmax = n // 2
    E = host(ctx.energy_spectrum(f, kmax))
    cx = np.array([0, 1, -1, 0, 0, 1, -1, 1, -1.0])
    cy = np.array([0, 0, 0, 1, -1, 1, -1, -1, 1.0])
    rho = fe.sum(1)
    ref = np.zeros(kmax + 1)
    k = np.fft.fftfreq(n, 1.0 / n)
    shell = np.floor(np.hypot(k[:, None], k[None, :]) + 0.5).astype(int)
    for c in (cx, cy):
        w = np.fft.fft2((fe * c[:, None, None]).sum(1) / rho) / n**2
        e = 0.5 * (np.abs(w) ** 2).mean(0)
        ref += np.bincount(shell.ravel(), e.ravel(), minlength=shell.max() + 1)[:kmax + 1]
    assert np.max(np.abs(E[:kmax + 1] - ref) / ref) < 1e-10
