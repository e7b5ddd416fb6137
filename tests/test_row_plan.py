"""How the row form's launches are planned: host code, no GPU."""
import pytest

import paper_2312_08728_amd as B
from gpu_util import GENERAL, NARROW, SPLIT, ONE_TRIP, BY_DIE, row_plan


@pytest.mark.parametrize("p,n,asked,G", [
    (9, 20_000, 0, 59), (30, 8_192, 0, 80), (62, 5_000, 0, 96), (71, 2_000, 0, 47), (122, 2_000, 0, 80), (950, 500, 0, 155),   # 12 KB of rows each
    (16, 768, 0, 4), (128, 1_536, 0, 32), (100, 600, 0, 20), (200, 4_096, 0, 256),
    (18, 100_000, 255, 255), (178, 777, 25, 25), (598, 50, 37, 37), (950, 2_000, 255, 255), (1026, 300, 37, 37),               # as asked
])
def test_steps_launched_one_by_one_do_not_follow_the_persistent_kernels_limits(p, n, asked, G):
    """The kernels of a persistent chain hold other numbers of rows, and take multiples of eight workgroups."""
    assert row_plan(p, n, asked, B.BMGD_CHAIN_LAUNCH)[:3] == (G, 512 if p > 512 and (p % 4 or p > 1024) else 1024, 0)


@pytest.mark.parametrize("p,n,asked,optimizer,G,kernel", [
    (1026, 300, 8, 0, 8, GENERAL), (1026, 300, 12, 0, 12, GENERAL), (1030, 600, 16, 0, 16, GENERAL), (2046, 300, 8, 0, 8, GENERAL),
    (1026, 96, 8, 0, 8, SPLIT), (1026, 97, 8, 0, 8, GENERAL), (1026, 192, 8, 3, 8, SPLIT), (1026, 193, 8, 3, 8, GENERAL),
    (1502, 400, 16, 0, 16, SPLIT), (1502, 401, 16, 0, 16, GENERAL), (1502, 592, 16, 1, 16, SPLIT), (1502, 593, 16, 1, 16, GENERAL),
    (1502, 7_165, 128, 0, 128, GENERAL), (1502, 12_000, 256, 0, 256, SPLIT), (1502, 600, 25, 0, 24, SPLIT), (1502, 600, 37, 0, 32, SPLIT),
    (1502, 141, 12, 3, 12, GENERAL), (1502, 120, 12, 3, 8, SPLIT), (1026, 1_789, 64, 0, 64, SPLIT),
    (1500, 300, 8, 0, 8, SPLIT), (2048, 20_000, 64, 0, 64, SPLIT), (2500, 300, 8, 0, 8, SPLIT),      # multiples of four: as ever
    (1502, 300, 7, 0, 7, GENERAL),
])
def test_wide_rows_that_are_no_multiple_of_four_take_the_kernel_that_is_faster(p, n, asked, optimizer, G, kernel):
    """Many rows a workgroup: the general kernel, on the workgroups asked for."""
    plan = row_plan(p, n, asked, optimizer=optimizer)
    assert plan[0] == G and plan[2] == kernel


@pytest.mark.parametrize("p,n,asked,G,exchange", [
    (16, 600, 255, 255, ONE_TRIP), (16, 600, 248, 248, BY_DIE), (16, 40_000, 0, 208, BY_DIE), (9, 600, 136, 136, BY_DIE), (16, 600, 128, 128, ONE_TRIP), (8, 600, 255, 255, ONE_TRIP), (17, 600, 128, 128, ONE_TRIP),
    (7, 600, 256, 256, ONE_TRIP),
])
def test_exchange_of_few_columns(p, n, asked, G, exchange):
    plan = row_plan(p, n, asked)
    assert plan[2:4] == (NARROW, exchange) and plan[0] == G
