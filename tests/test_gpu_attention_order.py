"""Causal passes of one sequence with more attention workgroups than compute units: their (query chunk, key split) items
are dealt out by length, so every row has to come out once whatever the order; and passes whose key splits are folded tile by
tile.  Against dense attention in 64 bits."""
import math

import pytest
import torch

import tidar_inputs as TI

pytestmark = pytest.mark.gpu

# shape, causal rows, mask rows, cached keys: 8 kv heads (one XCD each) with just more than 256 items, with 65 per XCD (a
# third round, chunks that straddle two query heads), with a ragged last chunk behind a cached prefix; 2 kv heads (four
# XCDs each) with key splits, padding on some of the XCDs, and mask rows
# (the last three: few workgroups but many key splits, whose partial results lie as query tiles: a last tile of 4 rows, of 12, tiles
# that straddle two heads, more than eight splits)
CASES = [("8b-shape", 1030, 0, 0), ("8b-shape", 2048, 16, 0), ("8b-shape", 1333, 7, 1001), ("1.5b-shape", 700, 0, 0),
         ("1.5b-shape", 1501, 16, 300), ("1.5b-shape", 2047, 0, 4000), ("small-gqa", 50, 0, 3000),
         ("small-gqa", 113, 5, 900), ("8b-shape", 25, 2, 2000)]


@pytest.mark.parametrize("name,nc,nm,L", CASES)
def test_causal_pass_matches_dense_attention(name, nc, nm, L):
    import paper_2511_08923_amd as T
    print(f"causal pass {name} nc={nc} nm={nm} L={L}", flush=True)
    sh = TI.SHAPES[name].with_layers(1)
    n_q, n_kv, hd, R = sh.n_q_heads, sh.n_kv_heads, sh.head_dim, nc + nm
    ctx = T.tidar_create(T.make_config(sh, T.TIDAR_BF16, max_k=16, max_batch=1))
    pps = (L + nc + 15) // 16 + 1
    g = torch.Generator(device="cuda").manual_seed(nc + L)

    def normal(*size):
        return torch.empty(*size, dtype=torch.bfloat16, device="cuda").normal_(generator=g)

    table = TI.shuffled_page_table(pps, pps + 3, seed=nc).view(1, pps).cuda()
    kp, vp = normal(1, pps + 3, n_kv, 16, hd), normal(1, pps + 3, n_kv, hd, 16)
    q, kn, vn = normal(1, R, n_q, hd), normal(1, R, n_kv, hd), normal(1, R, n_kv, hd)
    out = torch.full((1, R, n_q, hd), float("nan"), dtype=torch.bfloat16, device="cuda")
    pos = torch.arange(L, device="cuda")
    pk = kp[0][table[0, pos // 16].long(), :, pos % 16]
    pv = vp[0][table[0, pos // 16].long(), :, :, pos % 16]
    kv = T.tidar_kv_cache(kp.data_ptr(), vp.data_ptr(), table.data_ptr(), pps, pps + 3)
    ws = torch.empty(512 << 20, dtype=torch.uint8, device="cuda")
    T.tidar_hybrid_attention(ctx, kv, 0, 1, torch.tensor([L], dtype=torch.int32, device="cuda"), q, kn, vn, nc, 1 if nm else 0,
                             nm if nm else 1, nc, out, L, ws)
    torch.cuda.synchronize()
    T.tidar_destroy(ctx)
    r = torch.arange(R, device="cuda").view(R, 1)
    j = torch.arange(R, device="cuda").view(1, R)
    new = torch.where(r < nc, j <= r, torch.ones_like(j <= r))          # a mask row sees the causal rows and its block
    seen = torch.cat([torch.ones(R, L, dtype=torch.bool, device="cuda"), new], 1)
    for h in range(n_q):
        kh = h // (n_q // n_kv)
        k = torch.cat([pk[:, kh], kn[0, :, kh]]).double()
        v = torch.cat([pv[:, kh], vn[0, :, kh]]).double()
        s = q[0, :, h].double() @ k.t().contiguous() / math.sqrt(hd)
        want = s.masked_fill(~seen, -math.inf).softmax(-1) @ v
        got = out[0, :, h].double()
        # numerators and result rounded to bf16 (2^-9 each) of values that are O(1) at most
        assert torch.allclose(got, want, atol=1e-2, rtol=2e-2), (h, float((got - want).abs().max()))
