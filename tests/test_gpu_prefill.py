"""Several prompts of different length through one prefill pass: every sequence against the oracle (fp32) and against
itself prefilled alone (bf16), whatever shares the pass with it."""
import pytest
import torch

import tidar_inputs as TI
from oracle import tidar_oracle as O

pytestmark = pytest.mark.gpu

# one-token prompts, page boundaries, prompts longer than the pass (alone, in several passes) between short ones, a long one
# that fills the pass, so many short ones that the segment table is full, one long and many short ones
LENS = [([1, 1, 1], 64, 1), ([16, 1, 17, 33], 64, 4), ([40, 64, 24, 100, 5, 6], 64, 3), ([64, 1, 63, 2], 64, 4),
        ([3 + i % 5 for i in range(35)], 256, 2), ([200] + [4] * 12, 256, 4)]


@pytest.fixture(scope="module")
def T():
    import paper_2511_08923_amd as T
    assert torch.cuda.is_available()
    return T


def _prompts(sh, lens, seed):
    p = torch.zeros(len(lens), max(lens), dtype=torch.int32)
    for b, P in enumerate(lens):
        p[b, :P] = TI.make_prompt(sh, P, seed=seed + b)[0]
    return p


@pytest.mark.parametrize("lens,chunk,k", LENS)
@pytest.mark.parametrize("room", [True, False])
def test_fp32_prompts_together_match_the_oracle(T, lens, chunk, k, room):
    """room False: a workspace that holds a single sequence's passes only, so fewer prompts share a pass."""
    sh = TI.TINY
    w = TI.make_weights(sh, seed=1)
    eng = T.Engine(sh, w, dtype=T.TIDAR_F32, max_k=4, max_batch=len(lens), max_seq_len=224, prefill_chunk=chunk)
    if not room:
        eng.ws = torch.empty(T.tidar_workspace_bytes(eng.ctx, 1, k, 224), dtype=torch.uint8, device="cuda")
    prompts = _prompts(sh, lens, 300)
    model = O.OracleModel(sh, w)
    for want_logits in (True, False):
        first, lg = eng.prefill(prompts, k, want_logits=want_logits, prompt_len=lens)
        torch.cuda.synchronize()
        assert eng.prefix_len.tolist() == lens
        for b in (range(len(lens)) if want_logits else [0, len(lens) - 1]):
            st = model.new_state(224)
            d, want = model.prefill(st, [int(t) for t in prompts[b, :lens[b]]], k)
            assert first[b].tolist() == d, b
            if want_logits:
                assert float((lg[b].cpu().double() - want).abs().max()) < 1e-4, b
            for layer in range(sh.n_layers):
                kk, vv = eng.read_cache(layer, b, lens[b])
                assert float((kk.cpu().double() - st.k[layer][:lens[b]]).abs().max()) < 1e-4, b
                assert float((vv.cpu().double() - st.v[layer][:lens[b]]).abs().max()) < 1e-4, b
    eng.close()


@pytest.mark.parametrize("lens,chunk,k", LENS + [([515, 430, 344], None, 16), ([900, 7, 130], None, 8)])
def test_bf16_prompts_together_match_each_alone(T, lens, chunk, k):
    sh = TI.SMALL_GQA
    w = TI.make_weights(sh, seed=3, dtype=torch.bfloat16)
    make = lambda B: T.Engine(sh, w, dtype=T.TIDAR_BF16, max_k=16, max_batch=B, max_seq_len=960, prefill_chunk=chunk)
    many, one = make(len(lens)), make(1)
    prompts = _prompts(sh, lens, 400)
    _, lg = many.prefill(prompts, k, want_logits=True, prompt_len=lens)
    for b, P in enumerate(lens):
        _, want = one.prefill(prompts[b:b + 1, :P], k, want_logits=True)
        # the bf16 tolerance of the small models, for two results that may each be off by it
        assert float((lg[b] - want[0]).abs().max()) < 4e-2, b
        for layer in range(sh.n_layers):
            for got, ref in zip(many.read_cache(layer, b, P), one.read_cache(layer, 0, P)):
                assert torch.allclose(got.float(), ref.float(), atol=2e-2, rtol=2e-2), b
    many.close()
    one.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_prompts_together_sample_and_report_like_each_alone(T, dtype):
    """Sampled first tokens are keyed by sequence and position; a token id outside the vocabulary marks its own sequence."""
    sh = TI.TINY if dtype == "f32" else TI.SMALL_GQA
    w = TI.make_weights(sh, seed=1, dtype=torch.float32 if dtype == "f32" else torch.bfloat16)
    lens, k = [20, 33, 7], 4
    eng = T.Engine(sh, w, dtype=T.TIDAR_F32 if dtype == "f32" else T.TIDAR_BF16, max_k=k, max_batch=3, max_seq_len=64)
    prompts = _prompts(sh, lens, 500)
    mode = T.make_mode(sample=True, temperature=1.0, seed=9)
    first, lg = eng.prefill(prompts, k, mode, want_logits=True, prompt_len=lens)
    fused, _ = eng.prefill(prompts, k, mode, prompt_len=lens)
    for b, P in enumerate(lens):
        noisy = lg[b, 0].cpu().double() + torch.from_numpy(O.gumbel_noise(9, b, P, sh.vocab))
        top = noisy.topk(2).values
        if float(top[0] - top[1]) > 1e-3:
            assert int(first[b, 0]) == int(noisy.argmax()), b
        assert first[b, 1:].tolist() == lg[b, 2:].argmax(-1).tolist()
    assert torch.equal(first, fused)
    bad = prompts.clone()
    bad[1, 5] = sh.vocab + 3
    got, _ = eng.prefill(bad, k, mode, prompt_len=lens)
    assert eng.prefix_len.tolist() == [20, -1, 7] and got[1].tolist() == [-1] * k
    assert torch.equal(got[[0, 2]], first[[0, 2]])
    eng.close()
