"""Every form of the spectrum's passes against the oracle, with the tolerance of
test_gpu_spectrum.py: one, two and four lines per thread (few members and small grids take
fewer), prime sizes (k and n - k together), shells that add the
member groups up themselves and behind the separate fold, and all shells up to the corner."""
import numpy as np
import pytest

import oracle
from paper_2308_03972_amd import binding
from gpu_helpers import cuda, host, need_gpu, random_state, say
from test_gpu_spectrum import _close

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("n,m,storage", [(3, 1, 0), (3, 9, 0), (3, 4, 1), (4, 3, 1), (15, 4, 0),
                                         (16, 8, 0), (16, 9, 1), (31, 1, 0), (31, 2, 1), (31, 8, 0),
                                         (31, 64, 0), (60, 20, 0), (97, 3, 0), (100, 16, 1),
                                         (127, 33, 0), (251, 1, 0), (254, 5, 0), (257, 2, 0)])
def test_sizes_match_oracle(n, m, storage):
    say(f"spectrum sizes: {n}x{n} M={m} storage={storage}")
    rng = np.random.default_rng(n * 100 + m)
    ctx = binding.Context(n, n, m, 0.6, 0.1, [[0, 0]], 2, (0.1, 0.1), 2.0, 1.05, storage=storage)
    f = ctx.import_canonical(cuda(random_state(rng, m, n, n)))
    ref = oracle.member_mean_spectrum(host(ctx.export_canonical(f)))
    kmax = min(len(ref) - 1, n)
    got = host(ctx.energy_spectrum(f, kmax))
    _close(got, ref[:kmax + 1])
    np.testing.assert_array_equal(host(ctx.energy_spectrum(f, kmax)), got)
