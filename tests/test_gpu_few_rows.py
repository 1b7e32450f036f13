"""The GEMM of up to 32 rows: one and two row tiles, both column splits, fewer chunks of K than its LDS ring holds and more, odd
steps of 32, column tiles that are half there or not at all, against fp64."""
import pytest
import torch

import tidar_inputs as TI
from test_gpu_ops import _gemm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 15, 16, 17, 32])
@pytest.mark.parametrize("N,K", [(16, 32), (48, 96), (784, 192), (2064, 256), (144, 320), (6128, 608), (6144, 544), (6160, 2080),
                                 (16400, 96), (24560, 1056), (1536, 8960)])
def test_few_row_gemm_matches_fp64_matmul(M, N, K):
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
