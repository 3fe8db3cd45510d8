"""The merged launches of a cycle: observation operator and statistics of every problem of a
batch in one launch (groups of 32 problems: 33 of them, both routes and both storages), and
the reduction of the nodes' diagnostics records straight from the records (up to 4096
nodes) or in two passes.

Tolerances: a batch equals each problem's own run_cycle bit for bit; the diagnostics equal a
plain numpy reduction to 1e-12 (sums of at most 4225 positive terms in FP64).
"""
import numpy as np
import pytest
import torch

from paper_2308_03972_amd import binding
from gpu_helpers import cuda, host, need_gpu, random_state, say

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("storage", [binding.STORAGE_F64, binding.STORAGE_F32_DEV])
def test_batch_of_33_problems_equals_each_alone(storage):
    say(f"cycle launches: 33 problems, storage {storage}")
    rng = np.random.default_rng(11)
    shapes = [(12 + k % 3, 10 + k % 2, (8, 16, 32)[k % 3], 2 + k % 2, 1 + k % 2)
              for k in range(33)]   # nx, ny, members, nvar, route

    def contexts():
        r = np.random.default_rng(12)
        out = []
        for nx, ny, M, nvar, route in shapes:
            flat = r.choice(nx * ny, size=3, replace=False)
            pts = np.stack([flat % nx, flat // nx], axis=1).astype(np.int32)
            out.append(binding.Context(nx, ny, M, 0.55, 0.1, pts, nvar, (0.02,) * nvar, 5.0, 1.05,
                                       route=route, storage=storage))
        return out

    fe = [random_state(rng, M, ny, nx) for nx, ny, M, _, _ in shapes]
    yo = [cuda(0.03 * rng.standard_normal(3 * s[3])) for s in shapes]
    alone = []
    for c, f, y in zip(contexts(), fe, yo):
        s = c.import_canonical(cuda(f))
        c.run_cycle(s, 1, y)
        alone.append(host(s))
    ctxs = contexts()
    states = [c.import_canonical(cuda(f)) for c, f in zip(ctxs, fe)]
    batch = binding.Batch(ctxs, states, 1, dict(forecast_blocks=0, tile_rows=2, bucket_granularity=2,
                                                use_graph=1, analysis_queue=0, steps_per_launch=1))
    batch.run_cycle(yo)
    torch.cuda.synchronize()
    for a, s in zip(alone, states):
        np.testing.assert_array_equal(a, host(s))


@pytest.mark.parametrize("nx,ny", [(5, 7), (64, 64), (65, 65)])
def test_cycle_diagnostics_equal_a_plain_reduction(nx, ny):
    say(f"cycle launches: diagnostics of {nx} x {ny}")
    rng = np.random.default_rng(13)
    M = 6
    fe = random_state(rng, M, ny, nx)
    truth = 0.03 * rng.standard_normal((2, ny, nx))
    pts = np.array([[1, 2], [3, 4]], np.int32)
    ctx = binding.Context(nx, ny, M, 0.55, 0.1, pts, 2, (0.02, 0.02), 4.0, 1.05)
    f = ctx.import_canonical(cuda(fe))
    diag = torch.zeros(2 * binding.DIAG_LEN, dtype=torch.float64, device="cuda")
    ctx.run_cycle(f, 0, cuda(0.03 * rng.standard_normal(4)), cuda(truth), diag)
    d = host(diag).reshape(2, -1)
    after = host(ctx.export_canonical(f))
    cx = np.array([0, 1, -1, 0, 0, 1, -1, 1, -1.0])
    cy = np.array([0, 0, 0, 1, -1, 1, -1, -1, 1.0])
    for got, state in zip(d, (fe, after)):
        rho = state.sum(1)
        uv = np.stack([(state * c[:, None, None]).sum(1)
                       for c in (cx, cy)]) / rho
        mean = uv.mean(1)
        rmse = np.sqrt(((mean - truth) ** 2).sum(0).mean())
        spread = np.sqrt((((uv - mean[:, None]) ** 2).sum((0, 1)) / (M - 1)).mean())
        assert abs(got[0] - rmse) <= 1e-12 * rmse and abs(got[1] - spread) <= 1e-12 * spread
        assert got[2] == 0 and abs(got[3] - rho.min()) <= 1e-14 and abs(got[4] - rho.max()) <= 1e-14


def test_two_step_batch_of_half_block_ensembles_equals_each_alone():
    """FP32 ensembles that 32 does not divide run as two units of 16 members per block of the
    two-step batch: odd and even numbers of units, next to 32- and 64-member problems; bit for bit each problem's own run_cycle."""
    say("cycle launches: two units per block")
    shapes = [(14, 13, 16), (20, 19, 64), (9, 8, 32), (19, 12, 16)]  # 9 and 8 units of 16

    def contexts():
        return [binding.Context(nx, ny, M, 0.55, 0.1, np.array([[3, 4], [7, 2]], np.int32), 2,
                                (0.02, 0.02), 5.0, 1.05, storage=binding.STORAGE_F32_DEV)
                for nx, ny, M in shapes]

    rng = np.random.default_rng(14)
    fe = [random_state(rng, M, ny, nx) for nx, ny, M in shapes]
    yo = [cuda(0.03 * rng.standard_normal(4)) for _ in shapes]
    alone = []
    for c, f, y in zip(contexts(), fe, yo):
        s = c.import_canonical(cuda(f))
        c.run_cycle(s, 5, y)
        alone.append(host(s))
    ctxs = contexts()
    states = [c.import_canonical(cuda(f)) for c, f in zip(ctxs, fe)]
    batch = binding.Batch(ctxs, states, 5, dict(forecast_blocks=0, tile_rows=2, bucket_granularity=2,
                                                use_graph=1, analysis_queue=0, steps_per_launch=2))
    batch.run_cycle(yo)
    torch.cuda.synchronize()
    for a, s in zip(alone, states):
        np.testing.assert_array_equal(a, host(s))
