"""Forwards of up to four rows with many query heads on one K/V head: their rows fill four 32-row query tiles (from 25 heads
on) although they are few enough for the folded chain, whose O projection reads the attention's partial results itself."""
import pytest
import torch

import tidar_inputs as TI
from oracle import tidar_oracle as O

pytestmark = pytest.mark.gpu

TOL = 2e-2          # logits of the small bf16 models against the oracle with the same rounding points
SCORE_TOL = 4e-2    # a logit and a log-sum-exp


@pytest.fixture(scope="module")
def T():
    import paper_2511_08923_amd as T
    assert torch.cuda.is_available()
    return T


def _model(heads, std):
    sh = TI.ModelShape("many-heads", 2, 256, heads, 1, 128, 512, 512, False)
    w = TI.make_weights(sh, seed=3, dtype=torch.bfloat16, std=std)
    return sh, w, O.OracleModel(sh, w, bf16_faithful=True)


# three tiles, four with a last one of 4 rows, four full ones; five rows (the separate launches) on the other side of the chain
@pytest.mark.parametrize("heads", [24, 25, 32])
@pytest.mark.parametrize("P,k", [(1, 3), (2, 2), (3, 1), (2, 3)])
def test_prefill_of_a_few_rows(T, heads, P, k):
    print(f"prefill heads={heads} P={P} k={k}", flush=True)
    sh, w, model = _model(heads, 0.02)
    eng = T.Engine(sh, w, dtype=T.TIDAR_BF16, max_k=4, max_batch=1, max_seq_len=64)
    prompt = TI.make_prompt(sh, P, seed=7)
    _, lg = eng.prefill(prompt, k, want_logits=True)
    st = model.new_state(64)
    _, want = model.prefill(st, [int(t) for t in prompt[0]], k)
    err = float((lg[0].cpu().double() - want).abs().max())
    print(f"  max err {err:.2e} of logits with std {float(want.std()):.2f}", flush=True)
    eng.close()
    assert err < TOL


# a pass of four rows: the whole text, behind one pass, behind four of them (nine key splits), as two causal and two mask rows
@pytest.mark.parametrize("heads", [24, 25, 32])
@pytest.mark.parametrize("S,bl,chunk", [(4, 0, None), (20, 0, 16), (1028, 0, 256), (2, 2, None)])
def test_scoring_pass_of_four_rows(T, heads, S, bl, chunk):
    print(f"score heads={heads} S={S} bl={bl} chunk={chunk}", flush=True)
    sh, w, model = _model(heads, 0.05)
    eng = T.Engine(sh, w, dtype=T.TIDAR_BF16, max_k=4, max_batch=1, max_seq_len=1056, prefill_chunk=chunk)
    text = TI.make_prompt(sh, S, seed=80 + S)
    tl = [int(t) for t in text[0]]
    ar, diff, _ = eng.score(text, block_len=bl)
    want, want_diff = (model.score(tl), None) if bl == 0 else model.training_forward(tl, bl)[:2]
    err = float((ar[0, :S - 1].cpu().double() - want).abs().max())
    print(f"  max err {err:.2e}", flush=True)
    eng.close()
    assert err < SCORE_TOL
    if bl:
        assert float((diff[0].cpu().double() - want_diff).abs().max()) < SCORE_TOL
