"""The direct solver far beyond kappa = 2^52: observation errors so small that every
eigenvalue of S / a that the network determines lies beyond 2^55, where X^{-1/2} is below
1e-8 and a sum of shifted inverses that ends too early no longer follows it.

Compared are the analysis anomalies (member minus ensemble mean): sqrt(beta) dX on what the
network does not see, and what is left of it, 2^-28 and less, on what it does.  Tolerance: the
solvers and the reference perturb S by a few n eps of its norm, which moves the anomalies by
that times the ratio of its largest to its smallest non-zero eigenvalue; with every factor
taken at 16 the bound is 16 n 2^-53 ratio of the forecast anomalies' maximum, plus one rounding
of the populations and of the means on either side.
"""
import math

import numpy as np
import pytest

from paper_2308_03972_amd import binding
from gpu_helpers import cuda, host, need_gpu, random_state, say

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


DIRECT = [(2, 1, 16), (2, 9, 64), (2, 20, 64), (2, 24, 64), (2, 28, 64), (1, 20, 8), (1, 30, 24),
          (1, 40, 48), (1, 60, 56)]
# (the iterative solver, at cap 29, on the observation route: the ensemble route's takes the
# rounding of its zero eigenvalue, here beyond -a, for a failed solve)
ITERATIVE = [(2, 1, 16), (2, 9, 64), (2, 28, 64)]


@pytest.mark.parametrize("log2", [56, 62, 68, 90])
@pytest.mark.parametrize("route,p,M,cap", [(*c, 30) for c in DIRECT] + [(*c, 29) for c in ITERATIVE])
def test_anomalies_under_nearly_exact_observations(route, p, M, cap, log2):
    say(f"condition: route {route}, {p} points, {M} members, 2^{log2}, cap {cap}")
    n, beta = 11, 1.05
    rng = np.random.default_rng(500 + p + M)
    fe = random_state(rng, M, n, n)
    flat = rng.choice(n * n, size=p, replace=False)
    pts = np.stack([flat % n, flat // n], axis=1)
    probe = binding.Context(n, n, M, 0.55, 0.1, pts, 2, (1.0, 1.0), math.inf, beta, route=route)
    f = probe.import_canonical(cuda(fe))
    yf = probe.observe(f)
    y = host(yf)
    dy = y - y.mean(axis=0)
    # the eigenvalues of dY dY^T that count, and the error that puts the largest at 2^log2
    lam, Q = np.linalg.eigh(dy @ dy.T)
    seen = lam > 1e-12 * lam[-1]
    lam = np.where(seen, lam, 0.0)
    ratio = lam[-1] / lam[seen][0]
    a = (M - 1) / beta
    sigma = math.sqrt(lam[-1] / (a * 2.0 ** log2))
    ctx = binding.Context(n, n, M, 0.55, 0.1, pts, 2, (sigma, sigma), math.inf, beta, route=route)
    ctx.set_checks(max_sweeps=cap)
    yo = yf.mean(dim=0).contiguous()
    ctx.analyze(f, yf, yo)
    ctx.check()
    got = host(ctx.export_canonical(f))
    got = got - got.mean(axis=0)
    dx = fe - fe.mean(axis=0)
    W = (Q * np.sqrt(beta / (1.0 + lam / (sigma * sigma * a)))) @ Q.T
    want = np.tensordot(W, dx, axes=(0, 0))
    size = 2 * p if route == 2 else M
    tol = 16 * size * 2.0 ** -53 * ratio * np.abs(dx).max() + 8 * 2.0 ** -53 * np.abs(fe).max()
    err = np.abs(got - want).max()
    say(f"  eigenvalue ratio {ratio:.1f}, error {err:.1e} (bound {tol:.1e})")
    assert err < tol
