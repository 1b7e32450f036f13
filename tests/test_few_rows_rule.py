"""Split counts of the products of 5 to 32 rows: in column blocks of 64 no more workgroups than compute units, and in blocks of 128
where those have room for two splits only and do not nearly fill the chip."""
import pytest
import torch

import tidar_inputs as TI
from test_gemm_plan import planner
from test_gpu_ops import _gemm


def test_blocks_of_64_columns_stay_within_one_round():
    plan = planner()
    for N in list(range(16, 5441, 16)) + list(range(7376, 8193, 16)):
        for K in (512, 1536, 4096, 8960, 12288, 28672):
            p = plan(6, N, K, False)
            assert p.splits * ((N + 63) // 64) <= 256, (N, K)
            assert plan(32, N, K, False).splits == p.splits


@pytest.mark.parametrize("N,K,splits", [(2176, 12288, 6), (4480, 12288, 3), (5440, 12288, 3), (5456, 12288, 6), (6016, 12288, 5),
                                        (7360, 8192, 4), (7376, 8192, 2), (8192, 8192, 2), (8208, 8192, 4), (1536, 8960, 9),
                                        (2048, 1536, 3), (4096, 12288, 4), (6144, 4096, 4)])
def test_split_counts(N, K, splits):
    assert planner()(6, N, K, False).splits == splits


@pytest.mark.gpu
@pytest.mark.parametrize("M", [5, 16, 20, 32])
@pytest.mark.parametrize("N,K", [(2176, 2080), (5440, 2080), (5456, 2080), (7360, 1056), (7376, 2080), (8192, 2048), (8208, 1056)])
def test_both_column_splits_match_fp64_matmul(M, N, K):
    import paper_2511_08923_amd as T
    print(f"few-row gemm M={M} N={N} K={K}", flush=True)
    ctx = T.tidar_create(T.make_config(TI.SHAPE_8B.with_layers(1), T.TIDAR_BF16, max_k=16, max_batch=1))
    a = TI.make_normal((M, K), seed=M + K, dtype=torch.bfloat16)
    w = TI.make_normal((N, K), seed=N + K, dtype=torch.bfloat16, std=0.02)
    got = _gemm(T, ctx, a, w)
    T.tidar_destroy(ctx)
    want = (a.cuda().double() @ w.cuda().double().T).cpu()
    assert not torch.isnan(got).any()
    # fp32 sums of K products with a standard deviation of 0.02: far fewer than K roundings of at most 2^-24 of a partial
    # sum that stays below 8 of its standard deviations
    assert float((got.double() - want).abs().max()) < K ** 0.5 * 8 * 0.02 * K ** 0.5 * 2.0 ** -24
