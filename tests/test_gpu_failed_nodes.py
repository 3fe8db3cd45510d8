"""The count of failed solves is a count of nodes: a NaN in one member's observation reaches
the matrix of every node whose local set holds that observation, and lbmletkf_check reports
exactly those, for every layout of the solver (one, two and four nodes per wavefront)."""
import re

import numpy as np
import pytest

from paper_2308_03972_amd import binding
from gpu_helpers import cuda, need_gpu, random_state, say

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


# (route, members, variables, points a side, cut-off): up to four, two and one nodes per
# wavefront; ensembles of 4, 16, 32 and 48
@pytest.mark.parametrize("route,M,nvar,side,d_cut", [(2, 16, 2, 4, 5.0), (2, 64, 2, 4, 9.0),
                                                     (2, 64, 3, 4, 9.0), (2, 64, 3, 4, 11.0),
                                                     (2, 64, 2, 6, 7.5), (1, 4, 2, 4, 7.0),
                                                     (1, 16, 2, 4, 7.0), (1, 32, 2, 4, 7.0),
                                                     (1, 48, 2, 4, 7.0)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_every_failed_node_counts_once(route, M, nvar, side, d_cut, bad):
    say(f"failed nodes: route {route}, M {M}, nvar {nvar}, side {side}, d_cut {d_cut}, {bad}")
    n = 32
    rng = np.random.default_rng(6)
    step = n // side
    pts = np.array([(step * i + 3, step * j + 1) for j in range(side) for i in range(side)],
                   np.int32)
    ctx = binding.Context(n, n, M, 0.55, 0.1, pts, nvar, (0.02,) * nvar, d_cut, 1.05, route=route)
    f = ctx.import_canonical(cuda(random_state(rng, M, n, n)))
    yf = ctx.observe(f)
    yo = (yf.mean(dim=0) + 0.01).contiguous()
    yf[M // 2, nvar * 5] = bad
    ctx.analyze(f, yf, yo)
    with pytest.raises(binding.LbmLetkfError) as e:
        ctx.check()
    ys, xs = np.mgrid[0:n, 0:n]
    dx = np.minimum(abs(xs - pts[5, 0]), n - abs(xs - pts[5, 0]))
    dy = np.minimum(abs(ys - pts[5, 1]), n - abs(ys - pts[5, 1]))
    want = int((dx * dx + dy * dy < 4 * d_cut ** 2).sum())
    say(f"  {want} nodes: {e.value}")
    assert want in [int(v) for v in re.findall(r"\d+", str(e.value))]
