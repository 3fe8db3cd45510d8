"""The launches a gradient takes on either side of the sizes where they change: states between
observation times written by tiled launches or by single steps and pairs, whatever the route the
same bits as single steps; several reverse steps per launch or one (7e4 node-members for up to
five members, 2e4 for more), against the oracle's gradient with the tolerances of
test_gpu_adjoint.py (1e-11 of the gradient's scale, 1e-13 of J)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2308_03972_amd import binding
from gpu_helpers import cuda, host, need_gpu, random_state, say
from test_gpu_adjoint import _gpu_gradient, _oracle_gradient, _problem

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("nx,ny,M,storage", [(150, 140, 19, 0), (150, 141, 19, 0), (190, 180, 12, 0),
                                             (157, 160, 16, 1), (150, 141, 20, 1)])
def test_states_between_observations(nx, ny, M, storage):
    say(f"gradient routes: {nx}x{ny} M={M} storage={storage}")
    steps, times = 5, 3
    rng = np.random.default_rng(9)
    f0 = cuda(oracle.lbm_steps(random_state(rng, M, ny, nx), 1, 0.56, 0.1))
    ctx = binding.Context(nx, ny, M, 0.56, 0.1, [[1, 2], [nx // 2, 5]], 2, (0.1, 0.1), 2.0, 1.05,
                          storage=storage)
    f = ctx.import_canonical(f0)
    yo = cuda(0.02 * rng.standard_normal((times, 4)))
    work = ctx.adjoint_workspace(steps, times)
    Js, grads = [], []
    for k in range(3):   # kept, then (two forward sweeps in a row) recomputed
        J = ctx.misfit_forward(f, 0.1, steps, yo, work)
        if k == 1:
            continue
        Js.append(J.clone())
        grads.append([t.clone() for t in ctx.misfit_backward(f, 0.1, steps, yo, work)])
    assert torch.equal(Js[0], Js[1])
    for a, b in zip(*grads):
        assert torch.equal(a, b)
    # one interval: its states in the workspace are those of single steps, bit for bit
    whole = ctx.adjoint_workspace(steps, 1)
    J1 = float(ctx.misfit_forward(f, 0.1, steps, yo[:1].contiguous(), whole)[0])
    torch.cuda.synchronize()
    base = whole.ptr - whole.buffer.data_ptr()
    raw = whole.buffer[base:base + whole.nbytes]
    slot = (f.numel() * f.element_size() + 255) // 256 * 256
    st, found = f.clone(), 0
    for _ in range(steps):
        ctx.step(st, 1)
        want = st.reshape(-1).view(torch.uint8)
        found += any(torch.equal(raw[k * slot:k * slot + want.numel()], want)
                     for k in range(1 + 2 * (steps - 1)))
    assert found == steps
    ref = float(((host(ctx.observe(st)) - host(yo[0])) ** 2).sum())
    assert abs(J1 - ref) <= 1e-13 * ref


@pytest.mark.parametrize("m,ny,nx", [(5, 118, 118), (5, 119, 119), (6, 58, 57), (6, 58, 58)])
def test_reverse_steps_per_launch(m, ny, nx):
    say(f"gradient routes: reverse steps {nx} x {ny} x {m}")
    p = _problem(600 + m + nx, m, ny, nx, npts=4, nvar=2, n_times=2, s=3)
    J, (g, gcs), (g2, gcs2) = _gpu_gradient(p, repeat=2)
    Jr, gr, gcsr = _oracle_gradient(p)
    assert abs(J - Jr) <= 1e-13 * Jr
    assert np.max(np.abs(g - gr)) <= 1e-11 * np.max(np.abs(gr))
    assert abs(gcs - gcsr) <= 1e-11 * abs(gcsr)
    assert np.array_equal(g, g2) and gcs == gcs2
