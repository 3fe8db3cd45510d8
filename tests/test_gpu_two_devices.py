"""The launches that need more LDS than a kernel may take by default, from one process on every
GPU it sees: the permission is per device.  Needs two GPUs."""
import numpy as np
import pytest
import torch

from paper_2308_03972_amd import binding
from gpu_helpers import host, need_gpu, random_state, say

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()
    if torch.cuda.device_count() < 2:
        pytest.skip("one GPU")


@pytest.mark.parametrize("nx,ny,M,storage", [(40, 24, 5, 0), (64, 61, 8, 0), (90, 48, 24, 1),
                                             (128, 128, 16, 0), (64, 64, 64, 1)])
def test_forecast_and_gradient_on_each_device(nx, ny, M, storage):
    say(f"two devices: {nx}x{ny} M={M} storage={storage}")
    rng = np.random.default_rng(2)
    canon = random_state(rng, M, ny, nx)
    yo = 0.02 * rng.standard_normal((2, 4))
    outs = []
    for dev in range(2):
        with torch.cuda.device(dev):
            ctx = binding.Context(nx, ny, M, 0.56, 0.1, [[1, 2], [nx // 2, 5]], 2, (0.1, 0.1), 2.0,
                                  1.05, storage=storage)
            f = ctx.import_canonical(torch.from_numpy(canon).cuda())
            ctx.step(f, 12)
            work = ctx.adjoint_workspace(4, 2)
            y = torch.from_numpy(yo).cuda()
            ctx.misfit_forward(f, 0.1, 4, y, work)
            g, gc = ctx.misfit_backward(f, 0.1, 4, y, work)
            outs.append([host(f), host(g), host(gc)])
    for a, b in zip(*outs):
        np.testing.assert_array_equal(a, b)
