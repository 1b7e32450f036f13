"""The LM head of 33 to 288 rows over a wide vocabulary: five column tiles per workgroup, one pass (kernels_gemm_rows.hip).  Two to
nine row tiles, five chunks of K (odd), a last workgroup with one of its ten column tiles of 16.  (Longer K, and these sums
against those of the neighbouring kernels: test_gpu_row_class.py.)"""
import pytest
import torch

import tidar_inputs as TI
from test_gemm_plan import planner

SHAPE = TI.ModelShape("wide-vocab", 1, 160, 2, 1, 128, 96, 76816, False)


@pytest.fixture(scope="module")
def weights():
    return TI.make_weights(SHAPE, seed=4, dtype=torch.bfloat16)


def test_rows_reach_the_kernel():
    plan = planner()
    for rows in range(33, 289):
        assert plan(rows, SHAPE.vocab, SHAPE.d_model, True).wide == 3
    assert plan(160, 65536, 4096, True).wide == 3 and plan(161, 65536, 4096, True).wide == 1
    assert plan(272, 151936, 1536, True).wide == 3 and plan(272, 151936, 4096, True).wide == 1 and plan(289, 151936, 1536, True).wide == 1
    assert plan(100, 65536 - 128, SHAPE.d_model, True).wide != 3 and plan(32, SHAPE.vocab, SHAPE.d_model, True).wide != 3


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [33, 64, 65, 97, 129, 160, 161, 193, 225, 257, 288])
def test_logits_against_the_oracle(weights, rows):
    import paper_2511_08923_amd as T
    from oracle import tidar_oracle as O
    print(f"wide vocabulary, {rows} rows", flush=True)
    text = TI.make_prompt(SHAPE, rows, seed=6)
    eng = T.Engine(SHAPE, weights, dtype=T.TIDAR_BF16, max_k=1, max_batch=1, max_seq_len=rows + 16)
    ar, _, _ = eng.score(text)
    got = ar[0, :rows - 1].cpu().double()
    eng.close()
    want = O.OracleModel(SHAPE, weights, bf16_faithful=True).score([int(t) for t in text[0]])
    assert float((got - torch.as_tensor(want).double()).abs().max()) < 2e-2      # the bf16 tolerance of the small models


# 42 to 272 rows in two to nine row tiles; three sequences, so that causal rows stand in other row tiles than the first too
@pytest.mark.gpu
@pytest.mark.parametrize("B,k", [(1, k) for k in (6, 8, 9, 11, 13, 14, 15, 16)] + [(3, 5), (3, 8), (2, 11)])
@pytest.mark.parametrize("sample,beta", [(False, 1.0), (True, 1.0), (True, 0.5)])
def test_fused_reduction_equals_the_logits_path(weights, B, k, sample, beta):
    """The same step with and without logits: the epilogue's maxima and the reduction of the written logits choose the same
    tokens, bit for bit.  Only the causal rows up to the first wrong draft and one mask block show in a step's outputs, so the
    step is run with 1, 2, ..., k right drafts: every causal row and every block come up.  (A step's first next draft is the
    token its next causal row would have accepted.)"""
    import paper_2511_08923_amd as T
    print(f"wide vocabulary, {B} x k = {k}, sample {sample}, beta {beta}", flush=True)
    assert planner()(B * k * (k + 1), SHAPE.vocab, SHAPE.d_model, True).wide == 3
    eng = T.Engine(SHAPE, weights, dtype=T.TIDAR_BF16, max_k=k, max_batch=B, max_seq_len=128)
    mode = T.make_mode(sample=sample, temperature=1.0, seed=9, beta=beta)
    drafts, _ = eng.prefill(TI.make_prompt(SHAPE, 40, seed=2, batch=B), k, mode)
    length = eng.prefix_len.clone()
    drafts[:, 1:] = (drafts[:, 1:] + 1) % (SHAPE.vocab - 1)
    reached = set()
    while True:
        out = []
        for want_logits in (False, True):
            eng.prefix_len.copy_(length)
            a, acc, nxt, _ = eng.step(drafts, k, hint=64, mode=mode, want_logits=want_logits)
            out.append((a.tolist(), [acc[b, :int(a[b])].tolist() for b in range(B)], nxt.tolist()))
        assert out[0] == out[1]
        lens = out[0][0]
        reached |= {(b, n) for b, n in enumerate(lens)}
        if min(lens) == k:
            break
        for b, n in enumerate(lens):
            if n < k:
                drafts[b, n] = out[0][2][b][0]
    eng.close()
    # a wrong draft may be right by accident, once in a vocabulary
    assert len(reached) >= B * k - 1 and {(b, n) for b in range(B) for n in (1, k)} <= reached
