"""The reverse sweep's several-steps-per-launch form against the oracle's gradient: regions
larger than the lattice, ragged tiles, members that do not fill a block's, intervals of one
launch, of several and with a short one, and both sides of the size where single steps
take over (7e4 node-members).

Tolerance: as for the single steps (test_gpu_adjoint.py), 1e-11 of the gradient's scale:
the same partials in FP64 in another order over at most 26 steps.
"""
import numpy as np
import pytest

from gpu_helpers import need_gpu, say
from test_gpu_adjoint import _gpu_gradient, _oracle_gradient, _problem

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("m,ny,nx,s,times", [(1, 5, 7, 6, 2), (1, 33, 40, 13, 2), (5, 24, 40, 7, 3),
                                             (3, 50, 31, 2, 3), (10, 40, 32, 5, 2),
                                             (7, 48, 90, 4, 2), (16, 64, 64, 6, 1),
                                             (16, 66, 66, 3, 1), (18, 63, 62, 3, 1)])
def test_tiled_reverse_sweep_matches_oracle(m, ny, nx, s, times):
    say(f"adjoint tiles: {nx} x {ny} x {m}, {times} intervals of {s} steps")
    p = _problem(4000 + m + nx, m, ny, nx, npts=5, nvar=2, n_times=times, s=s)
    J, (g, gcs), (g2, gcs2) = _gpu_gradient(p, repeat=2)
    Jr, gr, gcsr = _oracle_gradient(p)
    assert abs(J - Jr) <= 1e-13 * Jr
    assert np.max(np.abs(g - gr)) <= 1e-11 * np.max(np.abs(gr))
    assert abs(gcs - gcsr) <= 1e-11 * abs(gcsr)
    assert np.array_equal(g, g2) and gcs == gcs2   # the same again from the same forward sweep
