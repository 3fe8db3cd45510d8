"""The direct solver's form with two nodes per wavefront (33 to 48 local observations)
against the oracle: both sizes filled and with a remainder, two and three variables, and
observation errors from well conditioned to several passes over the poles (9 x 9 nodes: the
last wavefront holds one).

Tolerance: that of test_gpu_direct.py, 16 l 2^-53 kappa of the increment's maximum and never
below 1e-9.
"""
import numpy as np
import pytest

from gpu_helpers import need_gpu, rel_max, say
from test_gpu_direct import _case

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("sigma", [3.0, 1e-1, 1e-2, 1e-4, 1e-6])
@pytest.mark.parametrize("p,nvar", [(17, 2), (11, 3), (20, 2), (21, 2), (15, 3), (24, 2)])
def test_pairs_of_nodes_against_the_oracle(p, nvar, sigma):
    say(f"direct solver, pairs: {p} points, {nvar} variables, sigma {sigma}")
    fe, got, ref, kappa = _case(9, 64, p, sigma, 2, 30, 1300 + p, nvar)
    tol = max(1e-9, 16 * nvar * p * 2.0 ** -53 * kappa)
    assert np.isfinite(got).all()
    assert rel_max(got - fe, ref - fe) < tol
