"""Multi-step forecast launches against single steps, bit for bit, at problems that reach every
shape of block the planner hands out (test_step_plans.py checks that they do)."""
import pytest
import torch

from paper_2308_03972_amd import binding
from gpu_helpers import need_gpu, say
from step_shapes import REACH

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("nx,ny,M,storage", REACH)
def test_every_block_shape_equals_single_steps(nx, ny, M, storage):
    say(f"step shapes {nx}x{ny} M={M} storage={storage}")
    gen = torch.Generator(device="cuda").manual_seed(nx + 7 * ny + M)
    force = 1e-4 * torch.randn(2, ny, nx, generator=gen, dtype=torch.float64, device="cuda")
    ctx = binding.Context(nx, ny, M, 0.53, 0.15, [[0, 0]], 2, (0.1, 0.1), 2.0, 1.05, mu=1e-3,
                          force=force, storage=storage)
    start = ctx.init_equilibrium(0.03 * torch.randn(M, 2, ny, nx, generator=gen,
                                                    dtype=torch.float64, device="cuda"))
    ctx.step(start, 1)
    ref = start.clone()
    states = []
    for _ in range(12):
        ctx.step(ref, 1)
        states.append(ref.clone())
    for n in (2, 3, 4, 5, 6, 8, 12):
        f = start.clone()
        ctx.step(f, n)
        assert torch.equal(f, states[n - 1]), n
