"""J evaluated again and again without a gradient leaves the states between observation times
unwritten (they would cost it up to half its time), a gradient in between has them written
again, and the values are the same bits in every order."""
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


@pytest.mark.parametrize("nx,ny,M,steps,times", [(40, 24, 5, 12, 1), (40, 24, 5, 12, 2),
                                                 (96, 90, 16, 12, 1), (31, 20, 3, 9, 4)])
def test_states_are_kept_for_gradients_only(nx, ny, M, steps, times):
    say(f"misfit alone: {nx}x{ny} M={M} steps={steps} times={times}")
    rng = np.random.default_rng(3)
    ctx = binding.Context(nx, ny, M, 0.56, 0.1, [[1, 2], [nx // 2, 5]], 2, (0.1, 0.1), 2.0, 1.05)
    f = ctx.import_canonical(cuda(oracle.lbm_steps(random_state(rng, M, ny, nx), 2, 0.56, 0.1)))
    yo = cuda(0.02 * rng.standard_normal((times, 4)))
    work = ctx.adjoint_workspace(steps, times)
    state = 8 * f.numel()

    def written():
        """States' worth of the workspace that a forward sweep writes."""
        work.buffer.fill_(0x55)
        J = ctx.misfit_forward(f, 0.1, steps, yo, work)
        torch.cuda.synchronize()
        return float(J[0]), float((work.buffer != 0x55).sum()) / state

    J, first = written()
    want = [t.clone() for t in ctx.misfit_backward(f, 0.1, steps, yo, work)]
    every = min(times, 2) * (steps - 1) + times      # two intervals' states, the checkpoints
    assert first > 0.98 * every
    assert written() == (J, first)                   # after a gradient: kept again
    for _ in range(2):                               # nobody used them: nothing kept
        Jk, more = written()
        assert Jk == J
        assert more < 0.75 * first
    got = ctx.misfit_backward(f, 0.1, steps, yo, work)
    for g, w in zip(got, want):
        assert torch.equal(g, w)
    assert written() == (J, first)
    for g, w in zip(ctx.misfit_backward(f, 0.1, steps, yo, work), want):
        assert torch.equal(g, w)
