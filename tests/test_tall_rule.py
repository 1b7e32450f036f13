"""Which of the products with many short shares of K go to the kernel that holds all row tiles: where column blocks of 128 x splits
are a multiple of eight only from seven row tiles on, elsewhere at any row count (what both sides of the line measure stands at the
rule)."""
import pytest

from test_gemm_plan import planner


@pytest.mark.parametrize("N,K,splits", [(1536, 8192, 8), (2560, 6144, 6), (3072, 5120, 5), (1280, 12288, 12), (2048, 7168, 7)])
def test_a_multiple_of_eight_stays_with_two_passes(N, K, splits):
    plan = planner()
    for M in range(33, 321, 7):
        p = plan(M, N, K, False)
        assert p.splits == splits and (p.wide == 2) == (M > 192), M


@pytest.mark.parametrize("N,K,splits", [(1536, 8960, 9), (1152, 11264, 11), (2304, 6144, 6)])
def test_the_others_go_there(N, K, splits):
    plan = planner()
    for M in range(33, 321, 7):
        p = plan(M, N, K, False)
        assert p.splits == splits and p.wide == 2, M
