"""The calls that a user of the library makes, at the sizes that they make them: verification and
plain decode steps, draft-side tree levels, and prompts.

Every model is one of `card_inputs.SHAPES` (or the small odd one below), at its own depth or at
fewer layers of the same widths.  A model's logits come back whole, and so does the state that a call
updates: both page pools of the KV cache.  Tokens do not: an arg-max of the logits that are returned
turns over where two of them nearly tie, at any change of rounding.
"""
import math

import torch

import card_inputs as ci
import paper_2508_04462_amd as card

# widths that are no multiples of the tiles, the vocabulary odd
ODD = ci.ModelShape("odd", 3, 512, 8, 2, 128, 1048, 3001, ctx=200, r=8)
MODELS = dict(ci.SHAPES, odd=ODD)


def _step(model, layers, ctx, r, temperature=0.0):
    return {"kind": "step", "model": model, "layers": layers, "ctx": ctx, "r": r, "temperature": temperature}


def _level(kind, model, layers, ctx, nodes, k, keep):
    return {"kind": kind, "model": model, "layers": layers, "ctx": ctx, "nodes": nodes, "k": k, "keep": keep}


def _prompt(model, layers, ctx, r):
    return {"kind": "prompt", "model": model, "layers": layers, "ctx": ctx, "r": r}


def listed():
    cases = {
        # the smallest model, its own context and row count: launch and hand-over latency
        "tiny r4": _step("tiny", 2, 128, 4),
        # plain decode of the draft-sized model
        "1b decode": _step("llama1b", 16, 1024, 1),
        # the benchmark's own workload
        "8b r8": _step("llama8b", 32, 1024, 8),
        # plain decode (every cache miss is such a step) at a sampling temperature, a context that ends inside a page
        "8b decode T1": _step("llama8b", 32, 2041, 1, 1.0),
        # the widest steps of the benchmark's sweep
        "qwen r32": _step("qwen7b", 28, 4096, 32),
        # a ragged row count and context between the two ends of that sweep
        "qwen r13": _step("qwen7b", 28, 1777, 13),
        # 70B widths (as many layers as let three such models share the card)
        "70b r8": _step("llama70b", 8, 2048, 8),
        # a long context, where attention is a large share
        "8b long": _step("llama8b", 4, 32700, 5),
        # one level of the draft's tree in one call, and the selection of the next level's nodes
        "level 32": _level("level", "llama1b", 16, 1000, 32, 8, 50),
        # a level of the larger of the two cache sizes in use: wider than one call, two lanes side by side
        "level 100": _level("wide", "llama1b", 16, 1024, 100, 8, 100),
        # a prompt and the first step behind it: of ordinary length on the 8B shape ...
        "8b prompt": _prompt("llama8b", 32, 1000, 8),
        # ... and a short one on the draft-sized model
        "1b prompt": _prompt("llama1b", 16, 203, 1),
    }
    return [dict(case, name=name) for name, case in cases.items()]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    model, most = rng.choice([("tiny", 2), ("odd", 3), ("llama1b", 16), ("llama1b", 16), ("llama8b", 32), ("llama8b", 32),
                              ("qwen7b", 28), ("qwen7b", 28), ("llama70b", 6)])
    layers = most if most < 4 else rng.randint(max(1, most // 4), most)
    # a context costs its prompt: long ones on few layers
    ctx = _log_uniform(rng, 1, max(256, min(16000, 80000 // layers)))
    what = rng.random()
    if what < 0.6:
        return _step(model, layers, ctx, rng.randint(1, rng.choice([1, 8, 16, 32])), rng.choice([0.0, 0.0, 0.0, 0.7, 1.0]))
    k = rng.randint(1, 16)
    if what < 0.7:
        nodes = rng.randint(1, 32)
        return _level("level", model, layers, ctx, nodes, k, rng.randint(1, 100))
    if what < 0.8:
        # (widths around the two cache sizes in use, 50 and 100, whose 32-row pieces are whole pages of the
        # cache: two calls that run side by side then write no page in common)
        nodes = rng.choice([rng.randint(49, 64), rng.randint(97, 128)])
        return _level("wide", model, layers, ctx, nodes, k, rng.randint(1, 100))
    # a prompt costs no more than the 8B one above: 1000 tokens on 32 of those layers
    elems = MODELS[model].weight_elems_per_layer() * layers
    full = MODELS["llama8b"].weight_elems_per_layer() * 32
    return _prompt(model, layers, _log_uniform(rng, 9, max(64, min(6000, int(800 * full / elems)))), rng.randint(1, 8))


# ---- inputs ---------------------------------------------------------------------------------------


def _shape(case):
    return MODELS[case["model"]].with_layers(case["layers"])


def _generator(seed, *stream):
    g = torch.Generator(device="cuda")
    g.manual_seed(hash((seed, 0x5EED) + stream) & 0x7FFFFFFFFFFFFFFF)
    return g


_LAYER = ("wq", "wk", "wv", "wo", "wg", "wu", "wd")


def _weight(shape, seed, name, layer):
    """N(0, 0.02^2) in bf16; norm gains around one in fp32."""
    g = _generator(seed, sum(ord(c) * 131 ** i for i, c in enumerate(name)), layer)
    if name.startswith("g_"):
        return 1.0 + 0.25 * (2.0 * torch.rand(shape.d_model, device="cuda", generator=g) - 1.0)
    d, f, v = shape.d_model, shape.d_ffn, shape.vocab
    rows, cols = {"embed": (v, d), "lm_head": (v, d), "wq": (shape.q_dim, d), "wk": (shape.kv_dim, d), "wv": (shape.kv_dim, d),
                  "wo": (d, shape.q_dim), "wg": (f, d), "wu": (f, d), "wd": (d, f)}[name]
    return torch.empty((rows, cols), dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02, generator=g)


def _tokens(shape, seed, stream, n):
    return torch.randint(0, shape.vocab, (n,), device="cuda", generator=_generator(seed, 7, stream)).tolist()


def _tree(case, seed):
    """The nodes of three levels (root, children, the measured level): tokens and parents per level."""
    shape, nodes = _shape(case), case["nodes"]
    mid = max(1, min(32, nodes // 3))
    levels = [(_tokens(shape, seed, 20, 1), [-1]), (_tokens(shape, seed, 21, mid), [0] * mid)]
    parents = torch.randint(0, mid, (nodes,), device="cuda", generator=_generator(seed, 8)).tolist()
    levels.append((_tokens(shape, seed, 22, nodes), parents))
    return levels


def _sigma(case, seed):
    return torch.rand(case["nodes"], device="cuda", generator=_generator(seed, 9)) * 0.5 + 0.01


def _target(case, seed, max_ctx, grid_wgs=0):
    shape = _shape(case)
    pages = (max_ctx + 15) // 16
    order = torch.randperm(pages, device="cuda", generator=_generator(seed, 6)).tolist()
    tgt = card.Target(shape, max_ctx, page_order=order, grid_wgs=grid_wgs, pool_fill=0)
    for name in ("embed", "lm_head", "g_final"):
        tgt.pack(name, 0, _weight(shape, seed, name, 0))
    for layer in range(shape.n_layers):
        for name in _LAYER + ("g_attn", "g_ffn"):
            tgt.pack(name, layer, _weight(shape, seed, name, layer))
    return tgt


class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.case, shape, ctx = case, _shape(case), case["ctx"]
    ctx_tokens = _tokens(shape, seed, 1, ctx)
    if case["kind"] in ("step", "prompt"):
        r = case["r"]
        s.tgt = _target(case, seed, ctx + 64)
        s.cand = torch.tensor(_tokens(shape, seed, 2, r), dtype=torch.int32, device="cuda")
        s.pending = int(s.cand[0])
        s.logits = torch.empty((r, shape.vocab), dtype=torch.float32, device="cuda")
        if case["kind"] == "prompt":
            s.tokens = ctx_tokens
        else:
            s.tgt.prefill(ctx_tokens)
            t = case["temperature"]
            s.sampling = card.CardSampling(t, seed & 0xFFFFFFFF) if t > 0 else None
        return s
    # a level of the draft's tree: the levels above it have been forwarded
    levels = _tree(case, seed)
    nodes, k = case["nodes"], case["k"]
    base = (ctx + 15) // 16 * 16
    wide = case["kind"] == "wide"
    # the slots that each level starts at: one behind the other, or on pages of their own
    starts = [base]
    for toks, _ in levels:
        end = starts[-1] + len(toks)
        starts.append((end + 15) // 16 * 16 if wide else end)
    s.tgt = _target(case, seed, starts[-1] + 32, grid_wgs=128 if wide else 0)
    s.tgt.prefill(ctx_tokens)
    mask_base, rows = ctx // 16 * 16, None
    words = (starts[-1] - mask_base + 31) // 32
    for depth, (toks, parents) in enumerate(levels):
        status, rows = card.card_tree_mask_level(rows, parents, starts[depth], ctx, mask_base, words)
        assert status == card.CARD_OK
        if depth < 2:
            s.tgt.draft_level(ctx, toks, [ctx + depth] * len(toks), starts[depth], rows, mask_base, k)
    first = starts[2]
    s.sigma = _sigma(case, seed)
    s.n_keep = min(case["keep"], nodes * k)
    s.next_tokens = torch.empty(s.n_keep, dtype=torch.int32, device="cuda")
    s.next_scores = torch.empty(s.n_keep, dtype=torch.float32, device="cuda")
    s.next_parents = torch.empty(s.n_keep, dtype=torch.int32, device="cuda")
    positions = [ctx + 2] * nodes
    if wide:
        s.tgt.enable_lanes(2)
        s.call = (ctx, levels[2][0], positions, first, rows, mask_base, k)
        return s
    s.toks = torch.tensor(levels[2][0], dtype=torch.int32, device="cuda")
    s.positions = torch.tensor(positions, dtype=torch.int32, device="cuda")
    signed = [[w - (1 << 32) if w >= 1 << 31 else w for w in row] for row in rows]
    s.mask = torch.tensor(signed, dtype=torch.int32, device="cuda")
    s.rows = card.CardTreeRows(s.toks.data_ptr(), s.positions.data_ptr(), first, s.mask.data_ptr(), words, mask_base)
    s.topk_tokens = torch.empty((nodes, k), dtype=torch.int32, device="cuda")
    s.topk_probs = torch.empty((nodes, k), dtype=torch.float32, device="cuda")
    s.logits = torch.empty((nodes, shape.vocab), dtype=torch.float32, device="cuda")
    return s


# ---- one pass -------------------------------------------------------------------------------------


def _ok(status, where):
    if status < 0:
        raise card.CardError(status, where)


def _pools(tgt):
    return {"k_cache": tgt.k_pages.view(torch.bfloat16), "v_cache": tgt.v_pages.view(torch.bfloat16)}


def run(state):
    s, case, tgt = state, state.case, state.tgt
    kind = case["kind"]
    if kind == "prompt":
        # (the first step's candidates are fixed, not the prompt's own arg-max: that may be a near tie)
        tgt.prefill(s.tokens)
        _ok(tgt.enqueue_verify(case["ctx"], s.pending, case["r"], s.logits, s.cand), "card_verify")
        return {"logits": s.logits, **_pools(tgt)}
    if kind == "step":
        _ok(tgt.enqueue_verify(case["ctx"], s.pending, case["r"], s.logits, s.cand, s.sampling), "card_verify")
        return {"logits": s.logits, **_pools(tgt)}
    nodes, k = case["nodes"], case["k"]
    stream = torch.cuda.current_stream().cuda_stream
    if kind == "wide":
        res = tgt.draft_level_wide(*s.call)
        topk_tokens, topk_probs = res["topk_tokens"], res["topk_probs"]
    else:
        topk_tokens, topk_probs = s.topk_tokens, s.topk_probs
        _ok(card.card_draft_level(tgt.cfg, tgt.packed, tgt.kv(-1), case["ctx"], s.rows, nodes, k, tgt.workspace, stream, topk_tokens,
                                  topk_probs, s.logits), "card_draft_level")
    _ok(card.card_cache_select(s.sigma, topk_tokens, topk_probs, nodes, k, s.n_keep, s.next_tokens, s.next_scores, s.next_parents,
                               stream), "card_cache_select")
    out = {"probs": topk_probs, "scores": s.next_scores, **_pools(tgt)}
    if kind == "level":
        out["logits"] = s.logits
    return out


# ---- what a pass cannot do without, and how exact it is -------------------------------------------


def work(case):
    shape, ctx = _shape(case), case["ctx"]
    layers, head = shape.n_layers * shape.weight_elems_per_layer(), shape.vocab * shape.d_model
    rows = case["nodes"] if "nodes" in case else case["r"]

    def forward(n, before, logits):
        """n rows behind `before` positions, the vocabulary head on `logits` of them: (bytes, flops)."""
        kv = 4 * shape.n_layers * shape.kv_dim
        return (2 * layers + (2 * head if logits else 0) + kv * (before + n) + 2 * n * shape.d_model,
                2.0 * n * layers + 2.0 * logits * head + 4.0 * shape.n_layers * shape.q_dim * n * (before + n / 2))

    b, f = forward(rows, ctx, rows)
    b += 0 if case["kind"] == "wide" else 4 * rows * shape.vocab
    if case["kind"] == "prompt":
        pb, pf = forward(ctx, 0, 1)
        b, f = b + pb, f + pf
    return {"bytes": b, "flops": f}


def tolerance(case):
    # What is left between two correct implementations: the order of fp32 sums, activations carried as
    # two bf16 halves (16 bits), and the few cache values that fall on the other side of a bf16 rounding.
    # Measured against 64 bits: 1e-4 (tiny) to 3.4e-3 (70B widths) for logits, 7e-3 for probabilities and
    # scores, which double the error of the logits that they come from.
    return {"rel": 0.02, "max": 0.25} if "nodes" in case else {"rel": 0.012, "max": 0.25}


def _rope(x, positions, theta):
    """x [n][heads][h]: half-split pairs."""
    h = x.shape[-1]
    inv = theta ** (-2.0 * torch.arange(h // 2, device="cuda", dtype=torch.float64) / h)
    ang = positions.to(torch.float64)[:, None] * inv[None, :]
    c, s = torch.cos(ang)[:, None, :], torch.sin(ang)[:, None, :]
    a, b = x[..., : h // 2], x[..., h // 2:]
    return torch.cat([a * c - b * s, b * c + a * s], dim=-1)


def _forward64(shape, seed, tokens, positions, n_tail, tail_mask):
    """Logits (64 bits) of the last n_tail rows of a decoder forward over all rows: every row but the
    tail sees its predecessors and itself, tail row i what tail_mask[i] says.  K and V are stored in bf16."""
    n, h, G = len(tokens), shape.head_dim, shape.n_q_heads // shape.n_kv_heads
    pos = torch.tensor(positions, device="cuda")
    w64 = lambda name, layer: _weight(shape, seed, name, layer).to(torch.float64)  # noqa: E731
    x = _weight(shape, seed, "embed", 0)[torch.tensor(tokens, device="cuda")].to(torch.float64)

    def norm(v, g):
        return v / torch.sqrt(v.square().mean(dim=-1, keepdim=True) + shape.rms_eps) * g

    for layer in range(shape.n_layers):
        last = layer + 1 == shape.n_layers
        xn = norm(x, w64("g_attn", layer))
        first = n - n_tail if last else 0  # the last layer's other rows only leave K and V behind
        k = _rope((xn @ w64("wk", layer).t()).view(n, -1, h), pos, shape.rope_theta)
        v = (xn @ w64("wv", layer).t()).view(n, -1, h)
        k, v = (t.to(torch.float32).to(torch.bfloat16).to(torch.float64) for t in (k, v))
        q = _rope((xn[first:] @ w64("wq", layer).t()).view(n - first, -1, h), pos[first:], shape.rope_theta) / math.sqrt(h)
        o = torch.empty((n - first, shape.n_q_heads, h), dtype=torch.float64, device="cuda")
        cut = n - n_tail
        block = max(16, (1 << 27) // (G * n))  # scores of a block of rows and one KV head: about 1 GiB
        for r0 in range(first, n, block):
            r1 = min(n, r0 + block)
            see = torch.arange(n, device="cuda")[None, :] <= torch.arange(r0, r1, device="cuda")[:, None]
            if r1 > cut:
                see[max(0, cut - r0):] = tail_mask[max(0, r0 - cut): r1 - cut]
            for kvh in range(shape.n_kv_heads):
                qh = q[r0 - first: r1 - first, kvh * G: (kvh + 1) * G].reshape(-1, h).contiguous()
                sc = (qh @ k[:, kvh].t().contiguous()).view(r1 - r0, G, n)
                sc.masked_fill_(~see[:, None, :], -math.inf)
                sc = torch.softmax(sc, dim=-1).view(-1, n)
                o[r0 - first: r1 - first, kvh * G: (kvh + 1) * G] = (sc @ v[:, kvh].contiguous()).view(r1 - r0, G, h)
        x = x[first:] + o.reshape(n - first, -1) @ w64("wo", layer).t()
        xn = norm(x, w64("g_ffn", layer))
        act = torch.nn.functional.silu(xn @ w64("wg", layer).t()) * (xn @ w64("wu", layer).t())
        x = x + act @ w64("wd", layer).t()
    return norm(x, w64("g_final", 0)) @ w64("lm_head", 0).t()


def exact(case, seed):
    shape, ctx = _shape(case), case["ctx"]
    tokens = _tokens(shape, seed, 1, ctx)
    none = {"k_cache": None, "v_cache": None}  # their layout is the library's own
    if case["kind"] in ("step", "prompt"):
        r = case["r"]
        tokens += _tokens(shape, seed, 2, r)
        see = torch.arange(ctx + r, device="cuda")[None, :] <= torch.arange(ctx, ctx + r, device="cuda")[:, None]
        return {"logits": _forward64(shape, seed, tokens, list(range(ctx + r)), r, see), **none}
    levels = _tree(case, seed)
    n_tree = sum(len(t) for t, _ in levels)
    see = torch.zeros((n_tree, ctx + n_tree), dtype=torch.bool)
    see[:, :ctx] = True
    positions, first, above = list(range(ctx)), 0, 0
    for depth, (toks, parents) in enumerate(levels):
        for i, p in enumerate(parents):
            if p >= 0:
                see[first + i] |= see[above + p]
            see[first + i, ctx + first + i] = True
        tokens, positions = tokens + toks, positions + [ctx + depth] * len(toks)
        above, first = first, first + len(toks)
    nodes, k = case["nodes"], case["k"]
    logits = _forward64(shape, seed, tokens, positions, n_tree, see.cuda())[-nodes:]
    probs = torch.softmax(logits, dim=-1).topk(k, dim=-1).values
    scores = (probs * _sigma(case, seed).to(torch.float64)[:, None]).flatten().topk(min(case["keep"], nodes * k)).values
    out = {"probs": probs, "scores": scores, **none}
    if case["kind"] == "level":
        out["logits"] = logits
    return out
