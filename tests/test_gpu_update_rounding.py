"""The update of the populations rounds once at their own size: the analysis increment
(here 1e-4 of the populations and below) is summed by itself and added at the end, whatever
the number of local observations.  Tolerance: the increment's own error is below 1e-3 of an ulp
of the largest population (1e-12 of it), so x_bar, its sum with the mean increment and the last
addition leave at most half an ulp each; the ensemble mean's error cancels up to sqrt(beta) - 1.
Two ulps."""
import math

import numpy as np
import pytest

from paper_2308_03972_amd import binding
from gpu_helpers import cuda, host, need_gpu, random_state, say

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("route,p,M", [(2, 4, 16), (2, 9, 64), (2, 16, 40), (2, 24, 64),
                                       (2, 32, 64), (1, 20, 24), (1, 40, 64)])
def test_update_rounds_once(route, p, M):
    say(f"update rounding: route {route}, {p} points, {M} members")
    n, beta, sigma = 10, 1.05, 1e-4
    rng = np.random.default_rng(40 + p + M)
    base = random_state(rng, 1, n, n)
    fe = base * (1.0 + 1e-4 * rng.standard_normal((M,) + base.shape[1:]))
    flat = rng.choice(n * n, size=p, replace=False)
    pts = np.stack([flat % n, flat // n], axis=1)
    ctx = binding.Context(n, n, M, 0.55, 0.1, pts, 2, (sigma, sigma), math.inf, beta, route=route)
    f = ctx.import_canonical(cuda(fe))
    yf = ctx.observe(f)
    y = host(yf)
    yo = y.mean(axis=0) + 0.3 * sigma * rng.standard_normal(2 * p)
    ctx.analyze(f, yf, cuda(yo))
    ctx.check()
    got = host(ctx.export_canonical(f)).astype(np.longdouble)
    # the weights in 64 bits, the sum with the populations in more
    a = (M - 1) / beta
    z = (y - y.mean(axis=0)) / sigma
    lam, Q = np.linalg.eigh(z @ z.T)
    lam = np.maximum(lam, 0.0)
    W = (Q * np.sqrt(beta / (1.0 + lam / a))) @ Q.T
    w = Q @ ((Q.T @ (z @ ((yo - y.mean(axis=0)) / sigma))) / (a + lam))
    xl = fe.astype(np.longdouble)
    mean = xl.mean(axis=0)
    dx = (xl - mean).astype(np.float64)
    inc = np.tensordot(W + w[:, None], dx, axes=(0, 0))
    err = np.abs(got - (mean + inc)).max(axis=(0, 2, 3))
    ulp = np.spacing(np.abs(fe).max(axis=(0, 2, 3)))
    say(f"  largest error in ulps per population: {[round(float(e / u), 2) for e, u in zip(err, ulp)]}")
    assert (err <= 2 * ulp).all()
