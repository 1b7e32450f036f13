"""The fp32 forwards of a few rows (norm, RoPE and SwiGLU folded into the GEMMs) and the first one beyond them, against the
oracle: prefill, steps, one-token steps, cache."""
import pytest
import torch

import tidar_inputs as TI
from oracle import tidar_oracle as O

pytestmark = pytest.mark.gpu

# (head dim, q heads, kv heads, d_model, d_ff, k, prompt): one and two pieces of 128 k and widths that are no multiple of
# them, head dimensions of two, four and eight column tiles and two that are not taken (48, 16), ragged row tiles, 240 and 256
# rows and more (272), a residual stream too wide (272), a head of more column blocks than the folded form takes
CASES = [(32, 4, 4, 128, 512, 4, 40, 272), (64, 4, 2, 144, 96, 3, 17, 272), (128, 3, 1, 256, 160, 1, 31, 272),
         (32, 8, 2, 240, 48, 5, 16, 272), (64, 2, 1, 208, 80, 15, 33, 272), (128, 4, 4, 256, 64, 8, 70, 272),
         (32, 2, 2, 48, 32, 16, 15, 272), (32, 2, 2, 64, 32, 3, 253, 272), (48, 4, 2, 128, 64, 3, 20, 272),
         (16, 4, 4, 64, 64, 2, 9, 272), (64, 2, 2, 272, 64, 4, 12, 272), (32, 2, 1, 96, 64, 4, 12, 16384)]


@pytest.fixture(scope="module")
def T():
    import paper_2511_08923_amd as T
    assert torch.cuda.is_available()
    return T


@pytest.mark.parametrize("hd,n_q,n_kv,d_model,d_ff,k,P,vocab", CASES)
def test_fp32_forwards_match_the_oracle(T, hd, n_q, n_kv, d_model, d_ff, k, P, vocab):
    sh = TI.ModelShape("t", 2, d_model, n_q, n_kv, hd, d_ff, vocab, False)
    w = TI.make_weights(sh, seed=d_model + hd, std=0.05)
    for i, lw in enumerate(w["layers"]):                    # gains that are not all one
        lw["attn_norm"] = 1 + 0.1 * TI.make_normal((d_model,), seed=10 + i)
        lw["ffn_norm"] = 1 - 0.1 * TI.make_normal((d_model,), seed=20 + i)
    w["final_norm"] = 1 + 0.1 * TI.make_normal((d_model,), seed=30)
    model = O.OracleModel(sh, w)
    eng = T.Engine(sh, w, dtype=T.TIDAR_F32, max_k=k, max_batch=1, max_seq_len=P + 4 * k + 16)
    prompt = TI.make_prompt(sh, P, seed=P)
    st = model.new_state(P + 4 * k + 16)
    want, lg_o = model.prefill(st, [int(t) for t in prompt[0]], k)
    first, lg = eng.prefill(prompt, k, want_logits=True)
    tol = 2e-5 * float(lg_o.abs().max().clamp(min=1.0)) * (d_model / 128) ** 0.5       # fp32 sums of d_model products
    assert float((lg[0].cpu().double() - lg_o).abs().max()) < tol and first[0].tolist() == want
    drafts = first
    for _ in range(2):
        a_o, _, nxt_o, lg_o = model.tidar_step(st, [int(t) for t in drafts[0]])
        a, _, nxt, lg = eng.step(drafts, k, hint=P + 3 * k, want_logits=True)
        assert float((lg[0].cpu().double() - lg_o).abs().max()) < tol
        assert int(a[0]) == a_o and nxt[0].tolist() == nxt_o
        drafts = nxt.clone()
    L = int(eng.prefix_len[0])
    for layer in range(sh.n_layers):
        for got, ref in zip(eng.read_cache(layer, 0, L), (st.k[layer][:L], st.v[layer][:L])):
            assert float((got.cpu().double() - ref).abs().max()) < tol
    eng.close()


def test_fp32_steps_of_sequences_that_do_not_fit_store_nothing(T):
    """The K/V stores of the folded RoPE keep the guards of the stand-alone kernel: a sequence beyond its page table and one
    with a page id outside the pool leave the cache as it was, the third sequence steps as it does alone."""
    sh, k, P = TI.TINY, 4, 40
    w = TI.make_weights(sh, seed=1)
    eng = T.Engine(sh, w, dtype=T.TIDAR_F32, max_k=k, max_batch=3, max_seq_len=64)
    prompts = torch.cat([TI.make_prompt(sh, P, seed=11 + b) for b in range(3)])
    first, _ = eng.prefill(prompts, k)
    eng.prefix_len[0] = 62
    eng.page_table[1, P // 16] = 10 ** 6
    before = (eng.k_pages.clone(), eng.v_pages.clone())
    a, _, _, lg = eng.step(first, k, hint=P, want_logits=True)
    assert a.tolist()[:2] == [0, 0] and int(a[2]) >= 1
    mine = torch.zeros(eng.n_pages, dtype=torch.bool, device="cuda")
    mine[eng.page_table[2].long()] = True
    for pages, was in zip((eng.k_pages, eng.v_pages), before):
        assert torch.equal(pages[:, ~mine], was[:, ~mine]) and not torch.equal(pages[:, mine], was[:, mine])
    one = T.Engine(sh, w, dtype=T.TIDAR_F32, max_k=k, max_batch=1, max_seq_len=64)
    one.prefill(prompts[2:], k)
    _, _, _, want = one.step(first[2:].contiguous(), k, hint=P, want_logits=True)
    assert torch.allclose(lg[2], want[0], atol=1e-5)
    one.close()
    eng.close()
