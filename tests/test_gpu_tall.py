"""The GEMM whose workgroups hold every row tile of a pass (kernels_gemm_tall.hip): which sizes reach it, and the sums."""
import pytest
import torch

import tidar_inputs as TI
from test_gemm_plan import planner
from test_gpu_ops import _gemm

# two to twelve row tiles (waves without a tile, with one less than the others), passes of 7 + 6, 7 + 7 and 8 + 7 row tiles, two
# and three column tiles per workgroup with columns left over, odd k steps of 32, a last split shorter than the others
SIZES = [(33, 24576, 1056), (96, 17920, 1536), (97, 17424, 1024), (160, 17920, 1056), (190, 24560, 1120), (256, 17296, 1056),
         (288, 24576, 1088), (340, 24576, 1056), (384, 22544, 1024), (416, 24576, 1024), (440, 24560, 1056), (480, 24576, 1056),
         (33, 4096, 12288), (96, 3072, 8192), (65, 4112, 8224), (72, 1536, 8960), (130, 1776, 9216), (272, 1536, 8960),
         (310, 2048, 8192), (320, 1552, 8736)]


@pytest.mark.parametrize("M,N,K", SIZES)
def test_sizes_reach_the_kernel(M, N, K):
    p = planner()(M, N, K, False)
    t = (M + 31) // 32
    assert p.wide == 2 and not p.rows and not p.mid
    assert p.m_chunks == (t + 11) // 12 and p.mt == -(-t // p.m_chunks) and p.nt == (3 if p.splits == 1 else 2)
    assert 180 <= -(-((N + 31) // 32) // p.nt) * p.splits <= 256


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", SIZES)
def test_tall_gemm_matches_fp64_matmul(M, N, K):
    import paper_2511_08923_amd as T
    print(f"tall gemm M={M} N={N} K={K}", flush=True)
    ctx = T.tidar_create(T.make_config(TI.SHAPE_8B.with_layers(1), T.TIDAR_BF16, max_k=16, max_batch=4))
    a = TI.make_normal((M, K), seed=M + K, dtype=torch.bfloat16)
    w = TI.make_normal((N, K), seed=N + K, dtype=torch.bfloat16, std=0.02)
    got = _gemm(T, ctx, a, w)
    T.tidar_destroy(ctx)
    want = a.cuda().double() @ w.cuda().double().T
    assert not torch.isnan(got).any()
    # fp32 sums of K products with a standard deviation of 0.02: far fewer than K roundings of at most 2^-24 of a partial
    # sum that stays below 8 of its standard deviations
    assert float((got.double() - want.cpu()).abs().max()) < K ** 0.5 * 8 * 0.02 * K ** 0.5 * 2.0 ** -24


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [33, 72, 160, 288, 340])
def test_swiglu_epilogue_in_a_step_of_the_wide_product(rows):
    """gate/up of 8960 features inside a scoring pass: the fused SwiGLU against the one of the oracle's arithmetic, by the
    log-probabilities of a one-layer model."""
    import paper_2511_08923_amd as T
    from oracle import tidar_oracle as O
    sh = TI.ModelShape("t", 1, 1536, 12, 2, 128, 8960, 1024, False)
    assert planner()(rows, 2 * sh.d_ff, sh.d_model, False).wide == (2 if rows <= 288 else 1)
    w = TI.make_weights(sh, seed=4, dtype=torch.bfloat16)
    text = TI.make_prompt(sh, rows, seed=6)
    eng = T.Engine(sh, w, dtype=T.TIDAR_BF16, max_k=1, max_batch=1, max_seq_len=rows + 16)
    ar, _, _ = eng.score(text)
    want = O.OracleModel(sh, w, bf16_faithful=True).score([int(t) for t in text[0]])
    got = ar[0, :rows - 1].cpu().double()
    eng.close()
    assert float((got - torch.as_tensor(want).double()).abs().max()) < 2e-2      # the bf16 tolerance of the small models
