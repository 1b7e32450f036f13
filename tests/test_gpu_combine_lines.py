"""Steps of many short sequences, whose key splits are folded row by row: row counts on both sides of the 480 from which the rows of
an output line share an XCD, multiples of the 64 rows that go round the XCDs and others, against the same sequences alone."""
import pytest
import torch

import tidar_inputs as TI
from test_attention_order import plan_and_order

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,k", [(40, 3), (41, 3), (48, 3), (32, 4), (25, 4), (256, 1)])
def test_steps_of_many_sequences_match_each_alone(B, k):
    import paper_2511_08923_amd as T
    print(f"step of {B} sequences, k={k}", flush=True)
    sh, L = TI.SMALL_GQA, 150
    w = TI.make_weights(sh, seed=5, dtype=torch.bfloat16)
    p, _ = plan_and_order(sh.n_kv_heads, sh.n_q_heads // sh.n_kv_heads, k, k * k, L + k + k * (k + 1), B=B)
    assert not p.tiled
    many = T.Engine(sh, w, dtype=T.TIDAR_BF16, max_k=k, max_batch=B, max_seq_len=L + 4 * k)
    one = T.Engine(sh, w, dtype=T.TIDAR_BF16, max_k=k, max_batch=1, max_seq_len=L + 4 * k)
    lens = [L - b % 7 for b in range(B)]
    prompts = torch.cat([TI.make_prompt(sh, L, seed=20 + b % 11) for b in range(B)])
    first, _ = many.prefill(prompts, k, prompt_len=lens)
    _, _, _, lg = many.step(first, k, hint=L + k, want_logits=True)
    for b in (0, 1, B // 2, B - 2, B - 1):
        one.prefill(prompts[b:b + 1, :lens[b]].contiguous(), k)
        _, _, _, want = one.step(first[b:b + 1].contiguous(), k, hint=L + k, want_logits=True)
        # the bf16 tolerance of the small models, for two results that may each be off by it
        assert float((lg[b] - want[0]).abs().max()) < 4e-2, b
    many.close()
    one.close()
