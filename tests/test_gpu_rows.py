"""GPU parity of the many-row GEMM (481 rows and more): pass heights, remainders, and its epilogues against each other."""
import math

import pytest
import torch

import tidar_inputs as TI
from test_gpu_ops import _gemm

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import paper_2511_08923_amd as T
    assert torch.cuda.is_available()
    return T


# row tiles as 9+7 .. 9+9 (two passes), 5s and 6s, a last pass that is one tile lower; one chunk of K, an odd count;
# a ragged column block, an odd 32-column tile, more workgroups than compute units
@pytest.mark.parametrize("M,N,K", [(481, 272, 32), (513, 784, 96), (545, 528, 64), (576, 1040, 1056), (608, 4112, 160),
                                   (650, 304, 608), (1665, 8208, 288), (2305, 256, 4096)])
def test_many_row_gemm_matches_fp64_matmul(T, M, N, K):
    print(f"many-row gemm M={M} N={N} K={K}", flush=True)
    ctx = T.tidar_create(T.make_config(TI.SHAPE_8B.with_layers(1), T.TIDAR_BF16, max_k=16, max_batch=4))
    a = TI.make_normal((M, K), seed=M + K, dtype=torch.bfloat16)
    w = TI.make_normal((N, K), seed=N + K, dtype=torch.bfloat16, std=0.02)
    got = _gemm(T, ctx, a, w)
    T.tidar_destroy(ctx)
    want = a.double() @ w.double().T
    assert not torch.isnan(got).any()
    # K products of size 0.02 summed in fp32: K * 2^-24 * 0.02 at the very worst, the bound of the other GEMM tests
    assert float((got.double() - want).abs().max()) < 2e-4 * max(1.0, math.sqrt(K / 256))


@pytest.mark.parametrize("sample,beta", [(False, 1.0), (True, 1.0), (True, 0.25)])
def test_many_row_step_fused_vocabulary_reduction_equals_logits_path(T, sample, beta):
    """Three sequences at k = 16 are 816 rows: without logits the LM head's epilogue reduces (and perturbs, or copies out
    for the mix) them in place, with logits they are written and reduced by the row kernel.  Same accumulators, same
    expressions: the tokens have to be the same."""
    sh, B, k, P = TI.SMALL_GQA, 3, 16, 40
    w = TI.make_weights(sh, seed=5, dtype=torch.bfloat16)
    eng = T.Engine(sh, w, dtype=T.TIDAR_BF16, max_k=k, max_batch=B, max_seq_len=160)
    mode = T.make_mode(sample=sample, temperature=1.0, seed=9, beta=beta)
    drafts, _ = eng.prefill(TI.make_prompt(sh, P, seed=6, batch=B), k, mode)
    drafts = drafts.clone()
    for _ in range(3):
        before = eng.prefix_len.clone()
        hint = int(before.max())
        with_logits = [t.cpu() for t in eng.step(drafts, k, hint=hint, mode=mode, want_logits=True)[:3]]
        eng.prefix_len.copy_(before)
        nxt = eng.step(drafts, k, hint=hint, mode=mode)
        fused = [t.cpu() for t in nxt[:3]]
        assert with_logits[0].tolist() == fused[0].tolist()
        for b in range(B):
            a = int(fused[0][b])
            assert with_logits[1][b, :a].tolist() == fused[1][b, :a].tolist()
        assert with_logits[2].tolist() == fused[2].tolist()
        drafts = nxt[2].clone()
    eng.close()


# kernels_gemm_mid: two to five and eight row tiles per pass with unequal passes, one k step per wave and fewer (K = 32:
# two of the four waves have none), a share of K that is no multiple of the ring, ragged N; wide single-split products
# up to five row tiles and beyond the eight-wave form
@pytest.mark.parametrize("M,N,K", [(33, 48, 32), (100, 784, 608), (272, 1536, 1536), (300, 1040, 96), (470, 2048, 1536),
                                   (480, 528, 288), (97, 16400, 160), (160, 24576, 608), (420, 24576, 96), (470, 24560, 512)])
def test_k_split_gemm_matches_fp64_matmul(T, M, N, K):
    test_many_row_gemm_matches_fp64_matmul(T, M, N, K)
