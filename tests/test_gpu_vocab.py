"""The LM head of 33 to 288 rows over a wide vocabulary: five column tiles per workgroup, one pass (kernels_gemm_rows.hip).  Two to
nine row tiles, five chunks of K (odd), a last workgroup with one of its ten column tiles of 16."""
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


@pytest.mark.gpu
@pytest.mark.parametrize("k", [6, 8, 9, 11, 13, 14, 15, 16])
@pytest.mark.parametrize("sample,beta", [(False, 1.0), (True, 1.0), (True, 0.5)])
def test_fused_reduction_equals_the_logits_path(weights, k, sample, beta):
    """The same step with and without logits: the epilogue's maxima and the reduction of the written logits choose the same
    tokens, bit for bit."""
    import paper_2511_08923_amd as T
    print(f"wide vocabulary, k = {k}, sample {sample}, beta {beta}", flush=True)
    eng = T.Engine(SHAPE, weights, dtype=T.TIDAR_BF16, max_k=k, max_batch=1, max_seq_len=128)
    mode = T.make_mode(sample=sample, temperature=1.0, seed=9, beta=beta)
    first, _ = eng.prefill(TI.make_prompt(SHAPE, 40, seed=2), k, mode)
    length = eng.prefix_len.clone()
    out = []
    for want_logits in (False, True):
        eng.prefix_len.copy_(length)
        a, acc, nxt, _ = eng.step(first, k, hint=64, mode=mode, want_logits=want_logits)
        out.append((int(a[0]), acc[0, :int(a[0])].tolist(), nxt[0].tolist()))
    eng.close()
    assert out[0] == out[1]
