"""RMSNorm of many rows (a wave per row): widths on both sides of what a lane holds and row counts that are no multiple of
the eight rows two workgroups share, by the log-probabilities of a one-layer model."""
import pytest
import torch

import tidar_inputs as TI
from oracle import tidar_oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_model,rows", [(32, 481), (544, 485), (1536, 527), (1568, 488), (2048, 543), (2080, 490), (4096, 483),
                                          (4128, 485)])
def test_scores_of_many_rows_match_the_oracle(d_model, rows):
    """4128: too wide for it."""
    import paper_2511_08923_amd as T
    sh = TI.ModelShape("t", 1, d_model, 2, 1, 128, 64, 512, False)
    w = TI.make_weights(sh, seed=d_model, dtype=torch.bfloat16)
    lw = w["layers"][0]
    lw["attn_norm"] = (1 + 0.2 * TI.make_normal((d_model,), seed=1)).to(torch.bfloat16)
    lw["ffn_norm"] = (1 - 0.2 * TI.make_normal((d_model,), seed=2)).to(torch.bfloat16)
    w["final_norm"] = (1 + 0.2 * TI.make_normal((d_model,), seed=3)).to(torch.bfloat16)
    text = TI.make_prompt(sh, rows, seed=rows)
    eng = T.Engine(sh, w, dtype=T.TIDAR_BF16, max_k=1, max_batch=1, max_seq_len=rows + 16)
    ar, _, _ = eng.score(text)
    want = O.OracleModel(sh, w, bf16_faithful=True).score([int(t) for t in text[0]])
    got = ar[0, :rows - 1].cpu().double()
    eng.close()
    assert float((got - torch.as_tensor(want).double()).abs().max()) < 2e-2      # the bf16 tolerance of the small models


@pytest.mark.parametrize("d_model,rows", [(32, 34), (4096, 66), (1536, 100), (4128, 72), (544, 480)])
def test_scores_of_a_few_hundred_rows_match_the_oracle(d_model, rows):
    """A workgroup per row, the rows of an output line on one XCD: row counts on both sides of whole lines and of the 64 rows
    that eight XCDs take in turn, a row wider than its threads' pieces (4128)."""
    test_scores_of_many_rows_match_the_oracle(d_model, rows)
