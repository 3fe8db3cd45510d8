"""The forecast planner on the host: every plan fits the kernel's limits, every split of a
forecast is one the planner priced, the shortest launches go where they are fastest, and the
problems of the bit-identity test reach every shape of block."""
import pytest

from step_shapes import MOST, REACH, planner, sample, shapes


def test_every_plan_fits_the_kernel():
    plans_of, launches_of = planner()
    for nx, ny, m, storage in sample(1500, 1):
        plans = plans_of(nx, ny, m, storage)
        elem = 4 if storage else 8
        per = 2 if storage and m % 2 == 0 else 1
        for n, mg, items in shapes(plans):
            p = plans.p[n]
            assert p.steps == n and mg % per == 0 and 1 <= mg <= m
            assert p.rx - 2 * (n - 1) >= 1 and p.ry - 2 * (n - 1) >= 1
            assert 9 * p.rx * p.ry * mg * elem <= 80 * 1024
            assert -(-(p.rx * p.ry * mg // per) // items) <= 1024
        if plans.most > 1:
            for steps in (2, 3, 4, 5, 7, 11, 20, 29):
                for even in (False, True):
                    k = launches_of(plans, steps, even)
                    assert 1 <= k <= steps and not (even and k % 2)
                    for n in {steps // k, -(-steps // k)}:
                        assert 1 <= n <= plans.most and plans.us[n] < 1e29


@pytest.mark.parametrize("nx,ny,m,storage,fewest",
                         [(512, 512, 50, 0, 2), (256, 256, 33, 0, 2), (200, 150, 24, 1, 2),
                          (512, 512, 14, 0, 2), (1024, 1024, 8, 0, 2), (90, 90, 9, 1, 2),
                          (61, 47, 3, 0, 2), (60, 50, 16, 0, 2), (512, 512, 16, 1, 3),
                          (256, 256, 1, 0, 1), (32, 32, 2, 0, 2), (512, 512, 2, 1, 1), (300, 300, 5, 0, 1),
                          (512, 512, 7, 0, 1), (1024, 1024, 8, 1, 1)])
def test_shortest_tiled_launch(nx, ny, m, storage, fewest):
    """Where two or three steps were slower as tiled launches than as single steps and pairs
    they are not taken, and where they were faster they are."""
    plans_of, _ = planner()
    plans = plans_of(nx, ny, m, storage)
    assert plans.most > 1 and plans.fewest == fewest


def test_bit_identity_cases_reach_every_shape():
    plans_of, _ = planner()
    have = {(s, mg, items) for nx, ny, m, s in REACH
            for _, mg, items in shapes(plans_of(nx, ny, m, s))}
    for nx, ny, m, s in sample(4000, 2):
        for n, mg, items in shapes(plans_of(nx, ny, m, s)):
            assert (s, mg, items) in have, (nx, ny, m, s, n, mg, items)
    assert max(n for nx, ny, m, s in REACH for n, _, _ in shapes(plans_of(nx, ny, m, s))) == MOST
