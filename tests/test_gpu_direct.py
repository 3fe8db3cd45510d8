"""The analysis' direct solver (tridiagonalisation and a sum of shifted inverses)
against the oracle and against the iterative Jacobi solver, which a sweep cap below
the default selects: every size with a remainder (unused rows, one and two matrix rows
per lane, a wavefront's last nodes missing), and observation errors that put the
condition number kappa = 1 + lambda_max / a of the transformed matrix in the first,
middle and last pole classes (one to six pole passes).

Tolerance: the tridiagonalisation and the oracle's eigensolver both perturb the l x l
matrix by a few l eps ||S||, which moves the increment by up to that times kappa / ||X||
relative; with every factor taken at 16 the bound is 16 l 2^-53 kappa of the
increment's maximum, never below the 1e-9 of the well-conditioned tests.
"""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2308_03972_amd import binding
from gpu_helpers import cuda, host, need_gpu, random_state, rel_max, say

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def _case(n, M, p, sigma, route, cap, seed, nvar=2):
    rng = np.random.default_rng(seed)
    fe = random_state(rng, M, n, n)
    flat = rng.choice(n * n, size=p, replace=False)
    pts = np.stack([flat % n, flat // n], axis=1)
    sig = (sigma,) * nvar
    ctx = binding.Context(n, n, M, 0.55, 0.1, pts, nvar, sig, math.inf, 1.05, route=route)
    ctx.set_checks(max_sweeps=cap)
    f = ctx.import_canonical(cuda(fe))
    yf = ctx.observe(f)
    yf_ref = oracle.observe(fe, pts, nvar)
    yo = yf_ref.mean(axis=0) + sigma * rng.standard_normal(nvar * p)
    ctx.analyze(f, yf, cuda(yo))
    ctx.check()
    ref = oracle.letkf_analysis(fe, yf_ref, yo, pts, sig, math.inf, 1.05)
    dy = (yf_ref - yf_ref.mean(axis=0)) / sigma
    kappa = 1.0 + np.linalg.norm(dy, 2) ** 2 * 1.05 / (M - 1)
    return fe, host(ctx.export_canonical(f)), ref, kappa


@pytest.mark.parametrize("cap", [30, 29])
@pytest.mark.parametrize("sigma", [3.0, 1e-2, 1e-4, 1e-6])
@pytest.mark.parametrize("route,p,M", [(2, 1, 9), (2, 4, 64), (2, 5, 33), (2, 8, 64), (2, 9, 64),
                                       (2, 12, 64), (2, 16, 64), (2, 20, 64), (2, 32, 64),
                                       (1, 6, 3), (1, 6, 8), (1, 6, 13), (1, 20, 16), (1, 6, 24),
                                       (1, 6, 31), (1, 6, 48), (1, 40, 64)])
def test_solvers_against_the_oracle(route, p, M, sigma, cap):
    say(f"direct solver: route {route}, {p} points, {M} members, sigma {sigma}, cap {cap}")
    fe, got, ref, kappa = _case(9, M, p, sigma, route, cap, 900 + p + M)
    n = 2 * p if route == 2 else M
    tol = max(1e-9, 16 * n * 2.0 ** -53 * kappa)
    err = rel_max(got - fe, ref - fe)
    say(f"  kappa {kappa:.1e} increment error {err:.1e} (bound {tol:.1e})")
    assert np.isfinite(got).all()
    assert err < tol


def test_batch_of_both_solvers_equals_each_problem_alone():
    """Three problems of one size, the middle one with a lowered sweep cap, in one
    batch (eager and as a work queue): each equals its own run_cycle bit for bit."""
    say("direct solver: batch with mixed sweep caps")
    rng = np.random.default_rng(77)
    pts = np.array([[3, 4], [9, 2], [6, 11], [12, 8], [1, 13]], dtype=np.int32)
    fe = [random_state(rng, 16, 14, 14) for _ in range(3)]
    yo = [cuda(0.03 * rng.standard_normal(10)) for _ in range(3)]

    def contexts():
        out = []
        for cap in (30, 12, 40):
            c = binding.Context(14, 14, 16, 0.55, 0.1, pts, 2, (0.01, 0.01), 6.0, 1.05, route=2)
            c.set_checks(max_sweeps=cap)
            out.append(c)
        return out

    alone = []
    for c, f, y in zip(contexts(), fe, yo):
        s = c.import_canonical(cuda(f))
        c.run_cycle(s, 3, y)
        alone.append(host(s))
    for queue in (0, 1):
        ctxs = contexts()
        states = [c.import_canonical(cuda(f)) for c, f in zip(ctxs, fe)]
        batch = binding.Batch(ctxs, states, 3, dict(forecast_blocks=0, tile_rows=2,
                                                    bucket_granularity=2, use_graph=1,
                                                    analysis_queue=queue))
        batch.run_cycle(yo)
        torch.cuda.synchronize()
        for a, s in zip(alone, states):
            np.testing.assert_array_equal(a, host(s))


@pytest.mark.parametrize("route,M,nvar,side", [(2, 64, 2, 4), (2, 64, 3, 4), (1, 40, 2, 4),
                                               (1, 16, 2, 4)])
def test_nan_observation_stays_at_its_nodes(route, M, nvar, side):
    """A NaN observation value reaches only the nodes whose local set holds it with a
    positive weight: all others -- in the same wavefront too, for one and several
    nodes per wavefront -- keep the clean analysis bit for bit, and no node counts as
    a failed solve (y^o does not enter the matrix)."""
    say(f"direct solver: NaN observation, route {route}, M {M}, nvar {nvar}")
    n = 32
    rng = np.random.default_rng(5)
    fe = random_state(rng, M, n, n)
    pts = np.array([(8 * i + 3, 8 * j + 1) for j in range(side) for i in range(side)], np.int32)
    d_cut = 8.0 if nvar == 3 else 7.0
    ctx = binding.Context(n, n, M, 0.55, 0.1, pts, nvar, (0.02,) * nvar, d_cut, 1.05, route=route)
    outs = []
    for bad in (False, True):
        f = ctx.import_canonical(cuda(fe))
        yf = ctx.observe(f)
        yo = (yf.mean(dim=0) + 0.01).contiguous()
        if bad:
            yo[nvar * 5] = float("nan")
        ctx.analyze(f, yf, yo)
        outs.append(host(ctx.export_canonical(f)))
    ctx.check()
    ys, xs = np.mgrid[0:n, 0:n]
    dx = np.minimum(abs(xs - pts[5, 0]), n - abs(xs - pts[5, 0]))
    dy = np.minimum(abs(ys - pts[5, 1]), n - abs(ys - pts[5, 1]))
    inside = dx * dx + dy * dy < 4 * d_cut ** 2
    assert not np.isfinite(outs[1][:, :, pts[5, 1], pts[5, 0]]).any()
    np.testing.assert_array_equal(outs[0][:, :, ~inside], outs[1][:, :, ~inside])
    assert np.isfinite(outs[0]).all()
