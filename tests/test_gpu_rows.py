"""GPU parity of the GEMM beyond 32 rows, kernel by kernel (pass heights, remainders, epilogues against each other), and of
what goes with it: fp32 GEMM and attention, the one-token step of many sequences."""
import math
from dataclasses import replace

import pytest
import torch

import tidar_inputs as TI
from test_gemm_plan import K_SPLIT, MANY_ROWS, TWO_PASS, WIDE
from test_gpu_ops import _attention_case, _gemm

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import paper_2511_08923_amd as T
    assert torch.cuda.is_available()
    return T


@pytest.mark.parametrize("M,N,K", MANY_ROWS)
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


# the vocabulary GEMM in passes of 6+5.. row tiles (816 rows), of 9+8 (544) and of 8+8 (504), the last column block ragged
@pytest.mark.parametrize("vocab,B,k", [(2048, 3, 16), (24560, 2, 16), (24560, 7, 8)])
@pytest.mark.parametrize("sample,beta", [(False, 1.0), (True, 1.0), (True, 0.25)])
def test_many_row_step_fused_vocabulary_reduction_equals_logits_path(T, sample, beta, vocab, B, k):
    """From 481 rows on: without logits the LM head's epilogue reduces (and perturbs, or copies out for the mix) them in
    place, with logits they are written and reduced by the row kernel.  Same accumulators, same expressions: the tokens
    have to be the same."""
    sh, P = replace(TI.SMALL_GQA, vocab=vocab), 40
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


@pytest.mark.parametrize("M,N,K", K_SPLIT + TWO_PASS + WIDE)
def test_gemm_of_33_to_768_rows_matches_fp64_matmul(T, M, N, K):
    test_many_row_gemm_matches_fp64_matmul(T, M, N, K)


# one (N, K) of each kernel family; row counts on both sides of every tile and pass arrangement of a class
@pytest.mark.parametrize("N,K,rows", [(16400, 608, (33, 72, 160, 161, 224, 272, 420, 480)),
                                      (784, 1056, (33, 97, 160, 161, 272, 350, 480)), (4096, 1056, (40, 160, 272, 480)),
                                      (784, 1056, (513, 640, 768)), (784, 1056, (769, 865, 1024)),
                                      (16400, 608, (545, 768)), (4096, 1056, (800, 1024))])
def test_a_rows_sum_does_not_follow_the_row_count(T, N, K, rows):
    """Bit for bit: what else is in flight (batch, k) must not move a row's result inside a row class."""
    ctx = T.tidar_create(T.make_config(TI.SHAPE_8B.with_layers(1), T.TIDAR_BF16, max_k=16, max_batch=4))
    a = TI.make_normal((rows[-1], K), seed=K, dtype=torch.bfloat16)
    w = TI.make_normal((N, K), seed=N, dtype=torch.bfloat16, std=0.02)
    most = _gemm(T, ctx, a, w)
    for M in rows[:-1]:
        assert torch.equal(_gemm(T, ctx, a[:M].contiguous(), w), most[:M]), (M, N, K)
    T.tidar_destroy(ctx)


# fp32: one element of everything, K that is no multiple of 32 or of 128, ragged rows (the narrow and the wide activation
# layout), more 16 x 16 tiles than the one-tile form takes
@pytest.mark.parametrize("M,N,K", [(1, 16, 8), (17, 48, 24), (20, 384, 128), (33, 80, 200), (272, 1040, 152)])
def test_fp32_gemm_matches_fp64_matmul(T, M, N, K):
    ctx = T.tidar_create(T.make_config(TI.TINY, T.TIDAR_F32, max_k=4, max_batch=1))
    a, w = TI.make_normal((M, K), seed=M + K).cuda(), TI.make_normal((N, K), seed=N + K, std=0.02).cuda()
    packed = torch.zeros(T.tidar_packed_weight_bytes(T.TIDAR_F32, N, K) // 4, device="cuda")
    T.tidar_pack_weight(T.TIDAR_F32, w, packed, N)
    out = torch.full((M, N), float("nan"), device="cuda")
    ws = torch.empty(T.tidar_gemm_workspace_bytes(T.TIDAR_F32, M, N, K), dtype=torch.uint8, device="cuda")
    T.tidar_gemm(ctx, a, packed, out, M, N, K, ws)
    err = (out.double() - a.double() @ w.double().T).abs().max()
    T.tidar_destroy(ctx)
    assert float(err) < K * 2.0 ** -24 * 0.02 * 16       # K roundings of sums that stay below 16 products of 0.02


def test_fp32_gemm_takes_buffers_at_any_float(T):
    """Packed weights and workspace one float past a 16-byte boundary: the same sums bit for bit."""
    M, N, K = 20, 80, 72
    ctx = T.tidar_create(T.make_config(TI.TINY, T.TIDAR_F32, max_k=4, max_batch=1))
    a, w = TI.make_normal((M, K), seed=1).cuda(), TI.make_normal((N, K), seed=2, std=0.02).cuda()
    got = []
    for off in (0, 1):
        packed = torch.zeros(T.tidar_packed_weight_bytes(T.TIDAR_F32, N, K) // 4 + off, device="cuda")[off:]
        T.tidar_pack_weight(T.TIDAR_F32, w, packed, N)
        ws = torch.empty(T.tidar_gemm_workspace_bytes(T.TIDAR_F32, M, N, K) // 4 + off, device="cuda")[off:]
        got.append(torch.full((M, N), float("nan"), device="cuda"))
        T.tidar_gemm(ctx, a, packed, got[-1], M, N, K, ws)
    T.tidar_destroy(ctx)
    assert torch.equal(got[0], got[1]) and not torch.isnan(got[0]).any()


# fp32 attention: head dimensions on both sides of 32 and 64 and one whose rows are no 16-byte pieces, several groups of
# four units per wave, several mask tiles
@pytest.mark.parametrize("hd,k,L", [(32, 4, 300), (64, 8, 70), (128, 16, 40), (128, 3, 270), (30, 5, 33), (96, 2, 0)])
def test_fp32_attention_head_dims(T, hd, k, L):
    sh = TI.ModelShape("t", 1, 128, 8, 8 if hd % 4 else 4, hd, 512, 512, False)
    for got, want in _attention_case(T, sh, 2, [L, max(L - 17, 0)], k, k, k, 1, seed=hd + L, dtype_id=T.TIDAR_F32):
        assert torch.allclose(got, want, atol=2e-5), float((got - want).abs().max())


@pytest.mark.parametrize("B", [5, 40])
def test_one_token_step_of_more_than_four_sequences(T, B):
    """The attention workgroups rotate the new rows at any batch: logits and the new K/V rows against the same sequence
    stepped alone (B = 40: more than 32 rows, the other GEMM class in front)."""
    sh = TI.SMALL_GQA
    w = TI.make_weights(sh, seed=5, dtype=torch.bfloat16)
    lens = [15 + 3 * (b % 13) for b in range(B)]           # page boundaries among them
    prompt = TI.make_prompt(sh, max(lens), seed=8, batch=B)
    tok = TI.make_drafts(sh, 1, seed=9, batch=B).view(B).cuda()
    many = T.Engine(sh, w, dtype=T.TIDAR_BF16, max_k=1, max_batch=B, max_seq_len=96)
    many.prefill(prompt, 1, prompt_len=lens)
    _, lg = many.ar_step(tok, hint=max(lens), want_logits=True)
    for b in (0, B // 2, B - 1):
        one = T.Engine(sh, w, dtype=T.TIDAR_BF16, max_k=1, max_batch=1, max_seq_len=96)
        one.prefill(prompt[b:b + 1, :lens[b]], 1)
        _, want = one.ar_step(tok[b:b + 1].contiguous(), hint=lens[b], want_logits=True)
        assert float((lg[b] - want[0]).abs().max()) < 2e-2          # the bf16 tolerance of the small models
        for layer in range(sh.n_layers):
            for got, ref in zip(many.read_cache(layer, b, lens[b] + 1), one.read_cache(layer, 0, lens[b] + 1)):
                assert torch.allclose(got.float(), ref.float(), atol=2e-2, rtol=2e-2)
        one.close()
    many.close()


@pytest.mark.parametrize("B", [3, 5, 20])
def test_swiglu_of_up_to_32_rows_divides(T, B):
    """silu(-88) is an ordinary fp32 number (-5.3e-37), but 1 / (1 + e^88) is below the smallest normal one, which an
    approximate reciprocal flushes to zero: the product with an `up` of 2^110 tells which was used.  Three rows: the
    GEMM that folds the norm in; five and twenty: one and two row tiles of the narrow one.  128 column blocks, one split."""
    sh = TI.ModelShape("t", 1, 256, 2, 1, 128, 8192, 512, False)
    w = TI.make_weights(sh, seed=3, dtype=torch.bfloat16)
    w["embed"] = torch.ones(sh.vocab, sh.d_model, dtype=torch.bfloat16)
    lw, f = w["layers"][0], torch.arange(sh.d_ff)
    for name in ("wo", "w_gate", "w_up", "w_down"):
        lw[name] = torch.zeros_like(lw[name])
    lw["w_gate"][f, f % sh.d_model] = -88.0
    lw["w_up"][f, f % sh.d_model] = 2.0 ** 110
    d = torch.arange(sh.d_model // 2)
    lw["w_down"][d, d] = 1024.0
    h = torch.tensor(-88.0 / (1.0 + math.exp(88.0)) * 2.0 ** 110).to(torch.bfloat16).double()      # -7e-4
    x = torch.ones(sh.d_model, dtype=torch.float64)
    x[d] += 1024.0 * h                                                                             # 0.29
    want = (x / x.pow(2).mean().sqrt()) @ w["lm_head"].double().T
    eng = T.Engine(sh, w, dtype=T.TIDAR_BF16, max_k=1, max_batch=B, max_seq_len=32)
    _, lg = eng.ar_step(torch.zeros(B, dtype=torch.int32, device="cuda"), hint=0, want_logits=True)
    err = float((lg.cpu().double() - want).abs().max())
    eng.close()
    assert err < 256 * 1.4 * 2.0 ** -9 * 0.02            # 256 products of |x| <= 1.4, rounded to 8 bits, and |w| ~ 0.02
