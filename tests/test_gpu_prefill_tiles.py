"""Prompts of different length in one pass whose key splits are folded tile by tile into the O projection's operand: last query
tiles that are not full, sequences with fewer tiles than the longest, against the oracle."""
import pytest
import torch

import tidar_inputs as TI
from oracle import tidar_oracle as O
from test_attention_order import plan_and_order

pytestmark = pytest.mark.gpu


# (query heads, kv heads, prompts, k): eight groups of a sequence and kv head or a multiple (dealt to XCDs) and other counts, two
# tiles against nine, last tiles of 4 to 30 rows and full ones, tiles that straddle two heads
@pytest.mark.parametrize("heads,kv,lens,k", [(8, 2, (61, 8, 35, 3), 4), (6, 1, (45, 13), 3), (16, 4, (30, 77), 2), (12, 2, (140, 6, 52), 8),
                                             (4, 1, (60, 28, 44), 4)])
def test_prompts_of_a_pass_match_the_oracle(heads, kv, lens, k):
    import paper_2511_08923_amd as T
    print(f"prefill heads={heads}/{kv} lens={lens} k={k}", flush=True)
    rows = [P + k for P in lens]
    p, _ = plan_and_order(kv, heads // kv, max(lens), k, max(rows), B=len(lens), segs=rows)
    assert p.tiled and p.splits > 1
    sh = TI.ModelShape("tiles", 2, 256, heads, kv, 128, 512, 512, False)
    w = TI.make_weights(sh, seed=3, dtype=torch.bfloat16)
    model = O.OracleModel(sh, w, bf16_faithful=True)
    eng = T.Engine(sh, w, dtype=T.TIDAR_BF16, max_k=k, max_batch=len(lens), max_seq_len=192)
    prompts = torch.zeros(len(lens), max(lens), dtype=torch.int32)
    for b, P in enumerate(lens):
        prompts[b, :P] = TI.make_prompt(sh, P, seed=90 + b)[0]
    _, lg = eng.prefill(prompts, k, want_logits=True, prompt_len=list(lens))
    torch.cuda.synchronize()
    errs = []
    for b, P in enumerate(lens):
        st = model.new_state(192)
        _, want = model.prefill(st, [int(t) for t in prompts[b, :P]], k)
        errs.append(float((lg[b].cpu().double() - want).abs().max()))
    print("  max errs " + " ".join(f"{e:.2e}" for e in errs), flush=True)
    eng.close()
    assert max(errs) < 2e-2              # the bf16 tolerance of the small models
