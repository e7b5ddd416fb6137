"""How the row form's launches are planned: host code, no GPU."""
import pytest

import paper_2312_08728_amd as B
from gpu_util import NARROW, ONE_TRIP, BY_DIE, row_plan


@pytest.mark.parametrize("p,n,asked,G", [
    (9, 20_000, 0, 59), (30, 8_192, 0, 80), (62, 5_000, 0, 96), (71, 2_000, 0, 47), (122, 2_000, 0, 80), (950, 500, 0, 155),   # 12 KB of rows each
    (16, 768, 0, 4), (128, 1_536, 0, 32), (100, 600, 0, 20), (200, 4_096, 0, 256),
    (18, 100_000, 255, 255), (178, 777, 25, 25), (598, 50, 37, 37), (950, 2_000, 255, 255), (1026, 300, 37, 37),               # as asked
])
def test_steps_launched_one_by_one_do_not_follow_the_persistent_kernels_limits(p, n, asked, G):
    """The kernels of a persistent chain hold other numbers of rows, and take multiples of eight workgroups."""
    assert row_plan(p, n, asked, B.BMGD_CHAIN_LAUNCH)[:3] == (G, 512 if p > 512 and (p % 4 or p > 1024) else 1024, 0)


@pytest.mark.parametrize("p,n,asked,G,exchange", [
    (16, 600, 255, 248, BY_DIE), (9, 600, 136, 136, BY_DIE), (16, 600, 128, 128, ONE_TRIP), (8, 600, 255, 255, ONE_TRIP), (17, 600, 128, 128, ONE_TRIP),
    (7, 600, 256, 256, ONE_TRIP),
])
def test_exchange_of_few_columns(p, n, asked, G, exchange):
    plan = row_plan(p, n, asked)
    assert plan[2:4] == (NARROW, exchange) and plan[0] == G
