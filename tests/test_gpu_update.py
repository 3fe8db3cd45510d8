"""The observation route's update (four nodes per wavefront, 16 lanes each) against the
oracle at the edges of its classes: members and local observations at and next to the
multiples of 16, one observation, odd ensembles, two and three variables, partly filled
wavefronts, and observations of weight zero on the rim of the localization.

Tolerance: well-conditioned problems (kappa below 1e3, at most 64 terms per sum), so the
1e-9 of the increment's maximum that the other FP64 analysis tests use.
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


@pytest.mark.parametrize("radius", [math.inf, 4.0])
@pytest.mark.parametrize("M,p,nvar", [(2, 1, 2), (7, 3, 2), (15, 5, 3), (16, 8, 2), (17, 8, 2),
                                      (32, 9, 2), (33, 16, 2), (48, 11, 3), (49, 17, 2),
                                      (63, 16, 3), (64, 24, 2), (64, 25, 2), (64, 32, 2)])
def test_update_against_the_oracle(M, p, nvar, radius):
    say(f"update: {M} members, {p} points, {nvar} variables, radius {radius}")
    nx = ny = 9  # 81 nodes: the last wavefront holds one
    rng = np.random.default_rng(7000 + 64 * M + p)
    fe = random_state(rng, M, ny, nx)
    flat = rng.choice(nx * ny, size=p, replace=False)
    pts = np.stack([flat % nx, flat // nx], axis=1).astype(np.int32)
    sig = (0.05,) * nvar
    ctx = binding.Context(nx, ny, M, 0.55, 0.1, pts, nvar, sig, radius, 1.05, route=2)
    f = ctx.import_canonical(cuda(fe))
    yf = ctx.observe(f)
    ref_yf = oracle.observe(fe, pts, nvar)
    yo = ref_yf.mean(axis=0) + 0.05 * rng.standard_normal(nvar * p)
    ctx.analyze(f, yf, cuda(yo))
    ctx.check()
    ref = oracle.letkf_analysis(fe, ref_yf, yo, pts, sig, radius, 1.05)
    got = host(ctx.export_canonical(f))
    assert np.isfinite(got).all()
    assert rel_max(got - fe, ref - fe) < 1e-9


def test_batch_of_member_classes_equals_each_problem_alone():
    """Problems of one eigenproblem size and 16, 32 and 64 members in one batch (eager and as
    a work queue): each equals its own run_cycle bit for bit."""
    say("update: batch of three member classes")
    pts = np.array([[3, 4], [9, 2], [6, 11], [12, 8], [1, 12]], dtype=np.int32)
    members = (32, 64, 16)

    def contexts():
        return [binding.Context(14, 13, M, 0.55, 0.1, pts, 2, (0.01, 0.01), 6.0, 1.05, route=2)
                for M in members]

    rng = np.random.default_rng(78)
    fe = [random_state(rng, M, 13, 14) for M in members]
    yo = [cuda(0.03 * rng.standard_normal(10)) for _ in members]
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
