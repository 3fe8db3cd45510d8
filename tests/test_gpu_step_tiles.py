"""Multi-step forecast launches against single steps, bit for bit: every shape of the
launch plan (1 to 8 members per block, regions of 16 to 24 nodes, one and two items per
thread, 2 to 6 steps per launch and the uneven splits in between), odd ensembles whose
last member group is short, ragged grids, grids smaller than the region (the halo wraps
around several times), with and without a force; and the sweeps that keep every
intermediate state, through the gradient."""
import numpy as np
import pytest
import torch

import oracle
from paper_2308_03972_amd import binding
from gpu_helpers import cuda, host, need_gpu, random_state, say

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("storage", [binding.STORAGE_F64, binding.STORAGE_F32_DEV])
@pytest.mark.parametrize("nx,ny,M", [(3, 3, 1), (5, 4, 2), (37, 23, 1), (150, 131, 1), (300, 217, 1),
                                     (17, 90, 2), (200, 181, 2), (33, 21, 3), (150, 147, 3),
                                     (40, 24, 5), (97, 61, 5), (230, 201, 5), (31, 29, 7),
                                     (32, 32, 8), (64, 61, 8), (129, 127, 8), (45, 44, 10),
                                     (23, 19, 16), (128, 117, 16), (150, 97, 20), (21, 20, 33),
                                     (41, 39, 50), (20, 17, 64)])
def test_many_steps_per_launch_equal_single_steps(nx, ny, M, storage):
    say(f"step tiles {nx}x{ny} M={M} storage={storage}")
    rng = np.random.default_rng(nx * 1000 + ny + M)
    canon = random_state(rng, M, ny, nx)
    force = cuda(1e-4 * rng.standard_normal((2, ny, nx))) if (nx + M) % 3 else None
    ctx = binding.Context(nx, ny, M, 0.53, 0.15, [[0, 0]], 2, (0.1, 0.1), 2.0, 1.05, mu=1e-3,
                          force=force, storage=storage)
    ref = ctx.import_canonical(cuda(canon))
    states = []
    for _ in range(13):
        ctx.step(ref, 1)
        states.append(ref.clone())
    for n in (2, 3, 5, 7, 12, 13):
        f = ctx.import_canonical(cuda(canon))
        ctx.step(f, n)
        assert torch.equal(f, states[n - 1]), n


@pytest.mark.parametrize("nx,ny,M,steps,storage", [(40, 24, 5, 7, 0), (33, 18, 1, 9, 0),
                                                   (30, 28, 12, 5, 1), (64, 64, 16, 4, 1)])
def test_gradient_over_multi_step_segments(nx, ny, M, steps, storage):
    """J of the multi-step sweeps against the misfit of the trajectory taken by single
    steps, and (FP64 storage) dJ/df0 along a random direction, whose reverse sweep reads
    every recomputed state, against central differences of J."""
    say(f"step tiles gradient {nx}x{ny} M={M} s={steps}")
    rng = np.random.default_rng(7)
    f0 = oracle.lbm_steps(random_state(rng, M, ny, nx), 2, 0.56, 0.1)
    pts = [[1, 2], [nx // 2, ny // 2], [nx - 1, 5]]
    ctx = binding.Context(nx, ny, M, 0.56, 0.1, pts, 2, (0.1, 0.1), 2.0, 1.05, storage=storage)
    yo = cuda(0.02 * rng.standard_normal((2, 6)))
    f = ctx.import_canonical(cuda(f0))
    work = ctx.adjoint_workspace(steps, 2)
    J = float(host(ctx.misfit_forward(f, 0.1, steps, yo, work))[0])
    g, gc = ctx.misfit_backward(f, 0.1, steps, yo, work)
    # the trajectory by single steps
    st, ref = f.clone(), 0.0
    for t in range(2):
        for _ in range(steps):
            ctx.step(st, 1)
        ref += float(((host(ctx.observe(st)) - host(yo[t])) ** 2).sum())
    assert abs(J - ref) <= 1e-13 * ref
    # dJ/df0 along a random direction, against central differences of the library's J in
    # FP64 storage (h^2 truncation and eps / h rounding below 1e-6 relative)
    if storage == 0:
        d = cuda(rng.standard_normal(f0.shape))
        h = 1e-6
        Js = [float(host(ctx.misfit_forward(ctx.import_canonical(cuda(f0) + s * h * d), 0.1, steps,
                                            yo, work))[0]) for s in (1, -1)]
        fd = (Js[0] - Js[1]) / (2 * h)
        got = float((g * d).sum())
        assert abs(got - fd) <= 1e-6 * max(abs(fd), float((g * g).sum().sqrt()))
