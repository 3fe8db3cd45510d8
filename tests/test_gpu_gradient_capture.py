"""A reverse sweep captured in a HIP graph, replayed between eager sweeps: the replay
recomputes the states between checkpoints into the same workspace, so an eager reverse sweep
after it must not take them for those the forward sweep left.  Every result equals, bit for
bit, the gradient of a context that never captured anything."""
import numpy as np
import pytest
import torch

import oracle
from paper_2308_03972_amd import binding
from gpu_helpers import cuda, need_gpu, random_state, say

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("nx,ny,M,steps,times", [(40, 24, 5, 7, 3), (20, 17, 3, 4, 5),
                                                 (16, 16, 16, 5, 2), (12, 10, 2, 3, 1),
                                                 (96, 96, 16, 6, 3)])
def test_replayed_reverse_sweep_between_eager_sweeps(nx, ny, M, steps, times):
    say(f"gradient capture {nx}x{ny} M={M} steps={steps} times={times}")
    rng = np.random.default_rng(11)
    f0 = cuda(oracle.lbm_steps(random_state(rng, M, ny, nx), 2, 0.56, 0.1))
    pts = [[1, 2], [nx // 2, ny // 2], [nx - 1, 5]]
    yo = cuda(0.02 * rng.standard_normal((times, 6)))

    def make():
        ctx = binding.Context(nx, ny, M, 0.56, 0.1, pts, 2, (0.1, 0.1), 2.0, 1.05)
        return ctx, ctx.import_canonical(f0), ctx.adjoint_workspace(steps, times)

    ctx, f, work = make()
    ctx.misfit_forward(f, 0.1, steps, yo, work)
    want = [t.clone() for t in ctx.misfit_backward(f, 0.1, steps, yo, work)]

    ctx, f, work = make()
    forward = lambda: ctx.misfit_forward(f, 0.1, steps, yo, work)
    backward = lambda: ctx.misfit_backward(f, 0.1, steps, yo, work)
    forward()
    backward()   # creates the recompute stream
    forward()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        captured = backward()

    def check(got, what):
        torch.cuda.synchronize()
        for g, w in zip(got, want):
            assert torch.equal(g, w), what

    check(backward(), "eager, after the capture")
    for k in range(3):
        forward()
        for t in captured:
            t.zero_()
        graph.replay()
        check(captured, f"replay {k}")
        check(backward(), f"eager after replay {k}")
        check(backward(), f"eager again after replay {k}")
        forward()
        check(backward(), f"forward and eager after replay {k}")
