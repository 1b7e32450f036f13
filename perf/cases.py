"""What the speed of this framework is judged by: calls of its public entry points as a decoding, serving or scoring
program makes them.

A case is a dict of plain values; `kind` says which entry point it goes through:

  step       Engine.step     one TiDAR decode step, batch x k(k+1) rows over a cached prefix
  ar         Engine.ar_step  the one-token step
  prefill    Engine.prefill  prompts into an empty cache, first drafts out
  score      Engine.score    log-probabilities of a text (block_len 0: causal section, else the training layout too)
  attention  tidar_hybrid_attention  the hybrid-mask attention of one layer on its own

Weights are drawn as everywhere in this repository (N(0, 0.02^2), norm gains 1), except that the embedding table is
wider and the LM head holds its rows one token further on.  A token's most likely successor is then the next id, by a
margin like a trained model's, and the drafts can be right up to a chosen length: steps accept as many tokens as the
paper's models do on average (about half of k), and which token wins is not decided by the last bit of a near tie.

`graph`: the program captured the step once and replays it, as decode loops do (bench.py among them); otherwise the
call launches from the host.  Every pass of a step starts from the same prefix length.
"""
import math

import torch

import paper_2511_08923_amd as T
import tidar_inputs as TI

DEV = "cuda:0"
PEAK = 200.0          # embedding rows are this much wider than N(0, 0.02^2): they stay visible through all layers


def _case(name, kind, shape, **more):
    c = {"kind": kind, "shape": shape, "dtype": "bf16", "batch": 1, "prefix": 0, "ragged": False, "k": 16,
         "sample": False, "beta": 1.0, "logits": False, "graph": False, "block_len": 0}
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call there is: the two-layer fp32 model, four drafts, every launch of it latency
        _case("tiny_fp32_step", "step", "tiny", dtype="f32", prefix=64, k=4, logits=True),
        # attention of one layer at the 8B head geometry, sixteen drafts over a 4096-token cache
        _case("attention_8b_k16", "attention", "8b-shape", prefix=4096),
        # plain decoding of a handful of sequences of different length on the small model, launched from the host
        _case("ar_1p5b_b6", "ar", "1.5b-shape", batch=6, prefix=1500, ragged=True),
        # the one-token step of the large model at batch 1: the latency the TiDAR step is compared with
        _case("ar_8b_b1", "ar", "8b-shape", prefix=4096, graph=True),
        # the small model's decode step after a short prompt, logits kept
        _case("step_1p5b_k16", "step", "1.5b-shape", prefix=701, logits=True, graph=True),
        # few drafts on a long context: 20 rows, the weight stream decides
        _case("step_8b_k4", "step", "8b-shape", prefix=8192, k=4, logits=True, graph=True),
        # the headline: batch 1, sixteen drafts, 4096 tokens of context
        _case("step_8b_k16", "step", "8b-shape", prefix=4096, graph=True),
        # a small sampled batch of sequences of different length, launched from the host (216 rows)
        _case("step_8b_b3_k8_sampled", "step", "8b-shape", batch=3, prefix=3000, ragged=True, k=8, sample=True),
        # a serving batch on long contexts: 2176 rows, the matrix cores decide
        _case("step_8b_b8_k16", "step", "8b-shape", batch=8, prefix=8192, ragged=True),
        # the long prompt of the large model
        _case("prefill_8b_4096", "prefill", "8b-shape", prefix=4096),
        # three short prompts of different length on the small model
        _case("prefill_1p5b_b3", "prefill", "1.5b-shape", batch=3, prefix=515, ragged=True, logits=True),
        # the training-layout forward over one text: causal section and mask section
        _case("score_1p5b_2000", "score", "1.5b-shape", prefix=2000, block_len=16),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "ar", "ar", "prefill", "prefill", "score", "attention", "tiny"])
    if kind == "tiny":
        return _case(None, "step", "tiny", dtype="f32", batch=rng.randint(1, 4), prefix=_log_int(rng, 16, 512),
                     k=rng.randint(1, 8), logits=True)
    shape = rng.choice(["1.5b-shape", "8b-shape"])
    if kind == "step":
        k = rng.choice([2, 3, 4, 6, 8, 8, 11, 13, 16, 16, 16])
        batch = _log_int(rng, 1, max(1, min(16, 2176 // (k * (k + 1)))))
        return _case(None, kind, shape, batch=batch, prefix=_log_int(rng, 64, 8192), ragged=batch > 1, k=k,
                     sample=rng.random() < 0.3, beta=rng.choice([1.0, 1.0, 1.0, 0.5]),
                     logits=batch * k * (k + 1) <= 600 and rng.random() < 0.4, graph=rng.random() < 0.5)
    if kind == "ar":
        batch = _log_int(rng, 1, 24)
        return _case(None, kind, shape, batch=batch, prefix=_log_int(rng, 64, 8192), ragged=batch > 1,
                     sample=rng.random() < 0.3, logits=rng.random() < 0.3, graph=rng.random() < 0.5)
    if kind == "prefill":
        batch = rng.randint(1, 3)
        return _case(None, kind, shape, batch=batch, prefix=_log_int(rng, 30, 2048 if shape == "8b-shape" else 4096) // batch + 1,
                     ragged=batch > 1, k=rng.choice([4, 8, 16]), logits=rng.random() < 0.5)
    if kind == "score":
        return _case(None, kind, shape, prefix=_log_int(rng, 60, 1500 if shape == "8b-shape" else 3000),
                     block_len=rng.choice([0, 0, 4, 7, 16]))
    k = rng.choice([4, 8, 11, 16])
    return _case(None, "attention", shape, batch=rng.randint(1, 4), prefix=_log_int(rng, 200, 8192), ragged=True, k=k)


# ---------------------------------------------------------------- inputs
def _lengths(case):
    """Prefix, prompt or text length of every sequence: all alike, or spread from a half to the whole of it."""
    B, P = case["batch"], case["prefix"]
    if not case["ragged"] or B == 1:
        return [P] * B
    return [max(1, P - i * P // (2 * B)) for i in range(B)]


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _weights(shape, seed, dtype):
    w = TI.make_weights(shape, seed, dtype=dtype, device=DEV)
    table = w["embed"]
    w["lm_head"] = table.roll(1, 0)          # row t+1 is what token t looks like at the end of the stack
    w["embed"] = table * PEAK
    return w


def _text(shape, B, S, seed):
    """Token ids that follow the model's own successor rule two times out of three."""
    g = _gen(seed)
    t = torch.randint(0, shape.vocab // 2, (B, S), generator=g, device=DEV, dtype=torch.int32)
    follow = torch.rand(B, S, generator=g, device=DEV) < 0.67
    pos = torch.arange(S, device=DEV, dtype=torch.int32).expand(B, S)
    start = torch.where(follow & (pos > 0), torch.zeros_like(pos), pos).cummax(1).values
    return ((t.gather(1, start.long()) + pos - start) % (shape.vocab - 1)).to(torch.int32).contiguous()


def _drafts(shape, B, k, seed):
    """Drafts that are right up to a seeded length (mean about half of k), wrong from there on."""
    c = TI.make_drafts(shape, 1, seed=seed, batch=B).to(torch.int64) % (shape.vocab // 2)
    keep = TI.make_acceptance_lengths(k, B, 1 + 0.483 * (k - 1), seed=seed + 1).to(torch.int64).view(B, 1)
    i = torch.arange(k).view(1, k)
    d = c + i + torch.where(i < keep, 0, 7)
    return d.to(torch.int32).to(DEV)


def _engine(case, shape, seed, max_batch, max_seq, max_k):
    bf16 = case["dtype"] == "bf16"
    w = _weights(shape, seed, torch.bfloat16 if bf16 else torch.float32)
    pps = (max_seq + T.PAGE - 1) // T.PAGE
    table = TI.shuffled_page_table(max_batch * pps, max_batch * pps, seed).view(max_batch, pps)
    return T.Engine(shape, w, dtype=T.TIDAR_BF16 if bf16 else T.TIDAR_F32, max_k=max_k, max_batch=max_batch,
                    max_seq_len=max_seq, page_table=table, device=DEV, free_source=True)


def _captured(body):
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        body()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        body()
    return graph


def prepare(case, seed):
    shape = TI.SHAPES[case["shape"]]
    kind, B, k = case["kind"], case["batch"], case["k"]
    lens = _lengths(case)
    st = {"case": case, "lens": lens}
    if kind == "attention":
        return _prepare_attention(case, shape, lens, seed, st)
    rows = {"step": k, "ar": 1, "prefill": k, "score": 0}[kind]
    eng = _engine(case, shape, seed, B, max(lens) + rows + T.PAGE, k if kind in ("step", "prefill") else 1)
    st["eng"] = eng
    st["mode"] = T.make_mode(sample=case["sample"], temperature=1.0, seed=seed + 3, beta=case["beta"])
    if kind in ("prefill", "score"):
        st["text"] = _text(shape, B, max(lens), seed + 5)
        return st
    # a decode loop somewhere in its run: the cache holds the prefix, the drafts are those of the last step
    g = _gen(seed + 7)
    for layer in range(shape.n_layers):
        eng.k_pages[layer].normal_(0.0, 1.0, generator=g)
        eng.v_pages[layer].normal_(0.0, 1.0, generator=g)
    st["len0"] = torch.tensor(lens, dtype=torch.int32, device=DEV)
    st["hint"] = max(lens) + rows
    if kind == "step":
        st["drafts"] = _drafts(shape, B, k, seed + 9)
        st["out"] = (torch.empty(B, dtype=torch.int32, device=DEV), torch.empty(B, k, dtype=torch.int32, device=DEV),
                     torch.empty(B, k, dtype=torch.int32, device=DEV))
    else:
        st["token"] = _drafts(shape, B, 1, seed + 9).view(B).contiguous()
        st["out"] = torch.empty(B, dtype=torch.int32, device=DEV)
    if case["graph"]:
        kept = []
        st["graph"] = _captured(lambda: kept.append(_decode(st)))
        st["kept"] = kept[-1]
    return st


def _prepare_attention(case, shape, lens, seed, st):
    B, k, hd = case["batch"], case["k"], shape.head_dim
    sh = shape.with_layers(1)
    ctx = T.tidar_create(T.make_config(sh, T.TIDAR_BF16, max_k=k, max_batch=B))
    pps = (max(lens) + k + T.PAGE - 1) // T.PAGE + 1
    R, g = k * (k + 1), _gen(seed)

    def normal(*size):
        return torch.empty(*size, dtype=torch.bfloat16, device=DEV).normal_(0.0, 1.0, generator=g)

    kp, vp = normal(1, B * pps, sh.n_kv_heads, 16 * hd), normal(1, B * pps, sh.n_kv_heads, 16 * hd)
    table = TI.shuffled_page_table(B * pps, B * pps, seed).view(B, pps).to(DEV)
    st.update(ctx=ctx, k_pages=kp, v_pages=vp, table=table, rows=R,
              kv=T.tidar_kv_cache(kp.data_ptr(), vp.data_ptr(), table.data_ptr(), pps, B * pps),
              q=normal(B, R, sh.n_q_heads, hd), k_new=normal(B, R, sh.n_kv_heads, hd),
              v_new=normal(B, R, sh.n_kv_heads, hd), out=normal(B, R, sh.n_q_heads, hd),
              len0=torch.tensor(lens, dtype=torch.int32, device=DEV), hint=max(lens),
              ws=torch.empty(512 << 20, dtype=torch.uint8, device=DEV))
    return st


# ---------------------------------------------------------------- one pass
def _decode(st):
    c, eng = st["case"], st["eng"]
    eng.prefix_len.copy_(st["len0"])
    if c["kind"] == "step":
        a, acc, nxt, lg = eng.step(st["drafts"], c["k"], hint=st["hint"], mode=st["mode"], want_logits=c["logits"],
                                   out=st["out"])
        got = {"accepted_len": a, "accepted": acc, "next_drafts": nxt}
    else:
        tok, lg = eng.ar_step(st["token"], hint=st["hint"], mode=st["mode"], want_logits=c["logits"], out=st["out"])
        got = {"token": tok}
    got["prefix_len"] = eng.prefix_len
    got["logits"] = lg
    got["k_pages"], got["v_pages"] = eng.k_pages, eng.v_pages
    return got


def run(st):
    c = st["case"]
    if c["kind"] in ("step", "ar"):
        if c["graph"]:
            st["graph"].replay()
            return st["kept"]
        return _decode(st)
    if c["kind"] == "prefill":
        eng = st["eng"]
        first, lg = eng.prefill(st["text"], c["k"], st["mode"], want_logits=c["logits"], prompt_len=st["lens"])
        return {"first_drafts": first, "logits": lg, "prefix_len": eng.prefix_len, "k_pages": eng.k_pages,
                "v_pages": eng.v_pages}
    if c["kind"] == "score":
        ar, diff, loss = st["eng"].score(st["text"], block_len=c["block_len"], length=st["lens"])
        return {"ar": ar, "diff": diff, "loss": loss, "k_pages": st["eng"].k_pages, "v_pages": st["eng"].v_pages}
    k = c["k"]
    T.tidar_hybrid_attention(st["ctx"], st["kv"], 0, c["batch"], st["len0"], st["q"], st["k_new"], st["v_new"], k, k, k,
                             1, st["out"], st["hint"], st["ws"])
    return {"out": st["out"], "k_pages": st["k_pages"], "v_pages": st["v_pages"]}


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    sh = TI.SHAPES[case["shape"]]
    kind, B, k, lens = case["kind"], case["batch"], case["k"], _lengths(case)
    es = 2 if case["dtype"] == "bf16" else 4
    per_layer = sh.d_model * (sh.q_dim + 2 * sh.kv_dim) + sh.q_dim * sh.d_model + 3 * sh.d_model * sh.d_ff
    head = sh.vocab * sh.d_model
    kv_row = 2 * sh.kv_dim * es                       # K and V of one token in one layer

    def step_keys(L):                                 # keys the rows of one step see, summed
        return k * L + k * (k + 1) // 2 + sum(k * (L + 1 + j + k) for j in range(k))

    if kind == "attention":
        R = k * (k + 1)
        keys = sum(step_keys(L) for L in lens)
        return {"bytes": sum(L * kv_row for L in lens) + B * R * (2 * sh.q_dim * es + kv_row),
                "flops": 4.0 * sh.q_dim * keys}
    if kind == "step":
        rows = head_rows = B * k * (k + 1)
        keys, kv_read, kv_write = sum(step_keys(L) for L in lens), sum(lens), B * k
    elif kind == "ar":
        rows = head_rows = B
        keys, kv_read, kv_write = sum(L + 1 for L in lens), sum(lens), B
    elif kind == "prefill":
        rows, head_rows = sum(L + k for L in lens), B * (1 + k)
        keys, kv_read, kv_write = sum(L * (L + 1) // 2 + k * (L + k) for L in lens), 0, sum(lens)
    else:
        bl = case["block_len"]
        rows = head_rows = sum(lens) * (2 if bl else 1)
        keys = sum(L * (L + 1) // 2 for L in lens)
        if bl:
            keys += sum(sum((i // bl) * bl + min(bl, L - (i // bl) * bl) for i in range(L)) for L in lens)
        kv_read, kv_write = 0, sum(lens)
    out = head_rows * sh.vocab * 4 if case["logits"] else head_rows * 4
    return {"bytes": float(es * (sh.n_layers * per_layer + head + rows * sh.d_model)
                           + sh.n_layers * kv_row * (kv_read + kv_write) + out),
            "flops": 2.0 * (rows * sh.n_layers * per_layer + head_rows * head) + 4.0 * sh.n_layers * sh.q_dim * keys}


def tolerance(case):
    """Measured by running every case with other split-K counts in its projections (sums in another order): the bf16
    rounding points turn differences of the fp32 sums into single flips of the last bit, layer after layer.  Seen:
    9.6e-3 in the logits of the 8B shape, 3.5e-3 in those of the 1.5B shape, 6e-2 of the rms for a single value."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.0}
    if case["kind"] == "attention":
        return {"rel": 4e-3, "max": 4e-2}
    return {"rel": 3e-2 if case["shape"] == "8b-shape" else 1.5e-2, "max": 0.24, "differ": 0.0}


# ---------------------------------------------------------------- the same in 64 bits
def _rows(kind, k, bl, L):
    """(position, causal keys seen, mask block or -1) of every row of one sequence, and how many of them are causal."""
    if kind == "step":
        rows = [(L + i, i + 1, -1) for i in range(k)] + [(L + 1 + j + s, j + 1, j) for j in range(k) for s in range(k)]
        return rows, k
    if kind == "ar":
        return [(L, 1, -1)], 1
    rows = [(i, i + 1, -1) for i in range(L)]
    if kind == "prefill":
        rows += [(L + s, L, 0) for s in range(k)]
    elif bl:
        rows += [(i, i // bl * bl, i // bl) for i in range(L)]
    return rows, L


def _seen(rows, nc, cached):
    """[rows, cached + rows]: which keys a row attends to."""
    vis = torch.tensor([r[1] for r in rows], device=DEV).view(-1, 1)
    blk = torch.tensor([r[2] for r in rows], device=DEV)
    i = torch.arange(len(rows), device=DEV)
    new = ((i < nc) & (i.view(1, -1) < vis)) | ((blk >= 0) & (blk == blk.view(-1, 1)))
    return torch.cat([torch.ones(len(rows), cached, dtype=torch.bool, device=DEV), new], 1)


def _attend(q, k, v, seen):
    """q [R, heads, hd], k and v [T, kv heads, hd], one kv head's group of query heads at a time."""
    R, nq, hd = q.shape
    out = torch.empty_like(q)
    group = nq // k.shape[1]
    for h in range(k.shape[1]):
        for i in range(h * group, (h + 1) * group):
            s = (q[:, i] @ k[:, h].t().contiguous()) / math.sqrt(hd)
            out[:, i] = s.masked_fill(~seen, -math.inf).softmax(-1) @ v[:, h].contiguous()
    return out


def _norm(x, gain, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * gain.double()


def _rotate(x, pos, base):
    half = x.shape[-1] // 2
    inv = base ** (-torch.arange(half, dtype=torch.float64, device=DEV) * 2 / x.shape[-1])
    ang = pos.double().view(-1, 1, 1) * inv
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], -1)


def _paged(kp, vp, table, L, hd):
    """K and V [L, kv heads, hd] of one sequence out of one layer's pages."""
    pos = torch.arange(L, device=DEV)
    page, slot = table[pos // T.PAGE].long(), pos % T.PAGE
    return (kp.view(kp.shape[0], kp.shape[1], T.PAGE, hd)[page, :, slot],
            vp.view(vp.shape[0], vp.shape[1], hd, T.PAGE)[page, :, :, slot])


def _place(kp, vp, table, L, k, v):
    pos = torch.arange(L, L + k.shape[0], device=DEV)
    page, slot, hd = table[pos // T.PAGE].long(), pos % T.PAGE, k.shape[-1]
    kp.view(kp.shape[0], kp.shape[1], T.PAGE, hd)[page, :, slot] = k
    vp.view(vp.shape[0], vp.shape[1], hd, T.PAGE)[page, :, :, slot] = v


def exact(case, seed):
    """What `run` returns, by the plain definition in 64 bits on the card (tokens and lengths: no such value)."""
    sh = TI.SHAPES[case["shape"]]
    kind, B, k, bl, lens = case["kind"], case["batch"], case["k"], case["block_len"], _lengths(case)
    hd = sh.head_dim
    if kind == "attention":
        st = _prepare_attention(case, sh, lens, seed, {})
        kp, vp, out = st["k_pages"][0].double(), st["v_pages"][0].double(), torch.empty_like(st["q"], dtype=torch.float64)
        for b, L in enumerate(lens):
            rows, nc = _rows("step", k, 0, L)
            kc, vc = _paged(kp, vp, st["table"][b], L, hd)
            kn, vn = st["k_new"][b].double(), st["v_new"][b].double()
            out[b] = _attend(st["q"][b].double(), torch.cat([kc, kn]), torch.cat([vc, vn]), _seen(rows, nc, L))
            _place(kp, vp, st["table"][b], L, kn[:nc], vn[:nc])
        return {"out": out, "k_pages": kp[None], "v_pages": vp[None]}
    new = {"step": k, "ar": 1, "prefill": k, "score": 0}[kind]
    pps = (max(lens) + new + T.PAGE + T.PAGE - 1) // T.PAGE
    size = (B * pps, sh.n_kv_heads, T.PAGE * hd)
    if sh.n_layers * math.prod(size) > 1 << 30:
        return None                                   # minutes and tens of gigabytes
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    w = _weights(sh, seed, dtype)
    table = TI.shuffled_page_table(B * pps, B * pps, seed).view(B, pps).to(DEV)
    cached = lens if kind in ("step", "ar") else [0] * B
    if kind == "step":
        toks = _drafts(sh, B, k, seed + 9)
    elif kind == "ar":
        toks = _drafts(sh, B, 1, seed + 9)
    else:
        toks = _text(sh, B, max(lens), seed + 5)
    g = _gen(seed + 7)
    xs, plan = [], []
    for b, L in enumerate(lens):
        rows, nc = _rows(kind, k, bl, L)
        ids = torch.cat([toks[b, :nc].long(), torch.full((len(rows) - nc,), sh.mask_token_id, device=DEV)])
        xs.append(w["embed"][ids].double())
        plan.append((nc, torch.tensor([r[0] for r in rows], device=DEV), _seen(rows, nc, cached[b])))
    k_pages, v_pages = [], []
    for lw in w["layers"]:
        m = {n: t.double() for n, t in lw.items()}
        kp, vp = torch.zeros(size, dtype=dtype, device=DEV), torch.zeros(size, dtype=dtype, device=DEV)
        if kind in ("step", "ar"):
            kp.normal_(0.0, 1.0, generator=g)
            vp.normal_(0.0, 1.0, generator=g)
        kp, vp = kp.double(), vp.double()
        for b, (nc, pos, seen) in enumerate(plan):
            x, L = xs[b], cached[b]
            h = _norm(x, m["attn_norm"], sh.rms_eps)
            q = _rotate((h @ m["wq"].t()).view(len(x), -1, hd), pos, sh.rope_base)
            kn = _rotate((h @ m["wk"].t()).view(len(x), -1, hd), pos, sh.rope_base)
            vn = (h @ m["wv"].t()).view(len(x), -1, hd)
            kc, vc = _paged(kp, vp, table[b], L, hd)
            x = x + _attend(q, torch.cat([kc, kn]), torch.cat([vc, vn]), seen).reshape(len(x), -1) @ m["wo"].t()
            h = _norm(x, m["ffn_norm"], sh.rms_eps)
            xs[b] = x + (torch.nn.functional.silu(h @ m["w_gate"].t()) * (h @ m["w_up"].t())) @ m["w_down"].t()
            _place(kp, vp, table[b], L, kn[:nc], vn[:nc])
        k_pages.append(kp)
        v_pages.append(vp)
    got = {"k_pages": torch.stack(k_pages), "v_pages": torch.stack(v_pages)}
    del k_pages, v_pages, m, lw
    w["layers"].clear()
    scored = kind == "score"
    if not (scored or case["logits"]):
        names = {"step": ("accepted_len", "accepted", "next_drafts", "prefix_len", "logits"),
                 "ar": ("token", "prefix_len", "logits"), "prefill": ("first_drafts", "logits", "prefix_len")}[kind]
        return {**{n: None for n in names}, **got}
    head = w["lm_head"].double()

    def logits(x):
        return _norm(x, w["final_norm"], sh.rms_eps) @ head.t()

    if scored:
        ar = torch.zeros(B, max(lens), dtype=torch.float64, device=DEV)
        diff = torch.zeros_like(ar) if bl else None
        for b, L in enumerate(lens):
            ids = toks[b, :L].long()
            for c in range(0, L, 512):
                e = min(c + 512, L - 1)
                if e > c:
                    ar[b, c:e] = logits(xs[b][c:e]).log_softmax(-1).gather(1, ids[c + 1:e + 1, None])[:, 0]
                if bl:
                    e = min(c + 512, L)
                    diff[b, c:e] = logits(xs[b][L + c:L + e]).log_softmax(-1).gather(1, ids[c:e, None])[:, 0]
        return {"ar": ar, "diff": diff, "loss": None, **got}
    if kind == "prefill":
        return {"first_drafts": None, "logits": torch.stack([logits(x[L - 1:]) for x, L in zip(xs, lens)]),
                "prefix_len": None, **got}
    lg = torch.stack([logits(x) for x in xs])
    if kind == "ar":
        return {"token": None, "prefix_len": None, "logits": lg[:, 0], **got}
    return {"accepted_len": None, "accepted": None, "next_drafts": None, "prefix_len": None, "logits": lg, **got}
