"""The coded copy of the weights gives the bits of the weights themselves: same blob, called with cfg.coded 1 and 0."""
import pytest
import torch

import card_inputs as ci

pytestmark = pytest.mark.gpu

SHAPES = {
    # widths that are no multiples of the tiles, three k-steps to a wavefront pair and fewer, a last k-step that is part zeros
    "odd": ci.ModelShape("odd", 2, 320, 5, 5, 64, 264, 1003, ctx=64, r=8),
    # heads of 128, tile counts that are multiples of four (grouped down-projection for more than eight rows)
    "wide": ci.ModelShape("wide", 2, 512, 4, 2, 128, 1416, 2050, ctx=64, r=8),
    # batches of more fragments than a word has bits, ending off a word's border: gate/up and the vocabulary head (8 tiles x 9 or 10 k-steps), the
    # down-projection (64 or 65) and the grouped one (4 tiles x 16 or 17)
    "long": ci.ModelShape("long", 2, 1216, 4, 2, 128, 8264, 2050, ctx=64, r=8),
}


def _weights(kind, rows, cols, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    w = torch.empty((rows, cols), device="cuda").normal_(0.0, 0.02, generator=g)
    if kind == "scales":  # every tensor in a range of its own
        w *= 2.0 ** ((seed * 7) % 9 - 6)
    elif kind == "spread":  # every weight needs its rest: exponents far apart, zeros and denormals among them
        e = torch.randint(-60, 1, w.shape, device="cuda", generator=g)
        w = torch.ldexp(w, e)
        w[:, ::5] = 0.0
        w[::7, 1::5] = 1e-40
    elif kind == "outliers":
        w[torch.rand(w.shape, device="cuda", generator=g) < 0.002] *= 300.0
    return w.to(torch.bfloat16)


def _pack(tgt, shape, kind, seed):
    d, f = shape.d_model, shape.d_ffn
    dims = {"wq": (shape.q_dim, d), "wk": (shape.kv_dim, d), "wv": (shape.kv_dim, d), "wo": (d, shape.q_dim), "wg": (f, d), "wu": (f, d),
            "wd": (d, f)}
    tgt.pack("embed", 0, _weights("normal", shape.vocab, d, seed))
    tgt.pack("lm_head", 0, _weights(kind, shape.vocab, d, seed + 1))
    tgt.pack("g_final", 0, torch.ones(d))
    for layer in range(shape.n_layers):
        for i, (name, (n, k)) in enumerate(dims.items()):
            tgt.pack(name, layer, _weights(kind, n, k, seed + 10 * layer + i + 2))
        for name in ("g_attn", "g_ffn"):
            tgt.pack(name, layer, torch.ones(d))


def _run(tgt, coded, r, n_ctx):
    """Logits of a step of r rows, candidates of a tree level of as many rows, and both page pools."""
    import paper_2508_04462_amd as card

    tgt.cfg.coded = coded
    toks = [(37 * i + 5) % tgt.cfg.vocab for i in range(n_ctx + r)]
    tgt.k_pages.zero_()
    tgt.v_pages.zero_()
    tgt.prefill(toks[:n_ctx], chunk=8)
    res = tgt.verify(n_ctx, -1, toks[n_ctx:], want_logits=True)
    assert res["accepted_len"] >= 0
    base, mask_base = n_ctx + r, n_ctx // 16 * 16
    st, rows = card.card_tree_mask_level(None, [-1] * r, base, n_ctx, mask_base, (base + r - mask_base + 31) // 32)
    assert st == card.CARD_OK
    lv = tgt.draft_level(n_ctx, toks[n_ctx:], [n_ctx] * r, base, rows, mask_base, 5)
    return [torch.as_tensor(x).contiguous().view(torch.uint8).cpu() for x in
            (res["logits"], lv["topk_tokens"], lv["topk_probs"], tgt.k_pages, tgt.v_pages)]


@pytest.mark.parametrize("grid_wgs", [0, 24, 5])  # one tile per workgroup at most; several batches; an odd grid
@pytest.mark.parametrize("kind", ["normal", "scales", "spread", "outliers"])
@pytest.mark.parametrize("name", sorted(SHAPES))
def test_coded_weights_give_the_same_bits(monkeypatch, name, kind, grid_wgs):
    import paper_2508_04462_amd as card
    from paper_2508_04462_amd import runtime

    monkeypatch.setattr(runtime, "CODED_MIN_LAYER_BYTES", 0)
    shape = SHAPES[name]
    tgt = card.Target(shape, 160, grid_wgs=grid_wgs, pool_fill=0)
    assert tgt.cfg.coded == 1
    tgt.packed.fill_(0xA5)  # nothing may depend on what the memory held
    # (weights packed over others leave nothing of them behind)
    _pack(tgt, shape, "spread" if kind == "normal" else "normal", 900)
    _pack(tgt, shape, kind, 50)
    for r in (1, 8, 13, 32):
        for got, want in zip(_run(tgt, 1, r, 41), _run(tgt, 0, r, 41)):
            assert torch.equal(got, want), (name, kind, grid_wgs, r)


def test_a_blob_without_the_copy_is_reported(monkeypatch):
    import paper_2508_04462_amd as card
    from paper_2508_04462_amd import runtime

    monkeypatch.setattr(runtime, "CODED_MIN_LAYER_BYTES", 0)
    shape = SHAPES["wide"]
    tgt = card.Target(shape, 160, pool_fill=0)
    tgt.packed.zero_()
    tgt.cfg.coded = 0
    _pack(tgt, shape, "normal", 3)
    assert tgt.verify(0, -1, [1, 2, 3])["accepted_len"] >= 0
    tgt.cfg.coded = 1
    assert tgt.verify(0, -1, [1, 2, 3])["accepted_len"] == -1


def _refused(tgt):
    """A step and a draft call both end at once: no token, nothing written to the cache."""
    tgt.k_pages.fill_(0x5A)
    res = tgt.verify(0, -1, [1, 2, 3])
    lv = tgt.draft_level(0, [1, 2], [0, 0], 0, [[1], [2]], 0, 3)
    return ((res["accepted_len"], res["correction_token"], res["kv_count"]) == (-1, -1, 0) and res["row_argmax"] == [-1] * 3
            and bool((lv["topk_tokens"] == -1).all()) and not bool(lv["topk_probs"].any()) and bool((tgt.k_pages == 0x5A).all()))


def test_weights_that_end_where_the_copy_would_begin_are_reported(monkeypatch):
    """Packed without the copy into a blob that has no room for one: the kernel must look before it streams."""
    import paper_2508_04462_amd as card
    from paper_2508_04462_amd import runtime

    monkeypatch.setattr(runtime, "CODED_MIN_LAYER_BYTES", 0)
    shape = SHAPES["wide"]
    tgt = card.Target(shape, 160, pool_fill=0)
    tgt.packed.fill_(0xFF)  # (as memory that held a blob with a copy may)
    whole = card.card_packed_weight_bytes(card.make_cfg(shape, 160))
    assert whole < tgt.packed.numel()
    tgt.packed = tgt.packed[:whole].clone()
    tgt.cfg.coded = 0
    _pack(tgt, shape, "normal", 3)
    assert tgt.verify(0, -1, [1, 2, 3])["accepted_len"] >= 0
    tgt.cfg.coded = 1
    assert _refused(tgt)
    tgt.cfg.coded = 0  # the same object keeps working
    assert tgt.verify(0, -1, [1, 2, 3])["accepted_len"] >= 0


@pytest.mark.parametrize("name,layer", [("wq", 0), ("wu", 1), ("wd", 4), ("lm_head", 0)])
def test_a_tensor_packed_without_its_copy_ends_the_copy(monkeypatch, name, layer):
    """... until that tensor is packed with it again, whatever else is packed in between."""
    import paper_2508_04462_amd as card
    from paper_2508_04462_amd import runtime

    monkeypatch.setattr(runtime, "CODED_MIN_LAYER_BYTES", 0)
    shape = SHAPES["odd"].with_layers(5)
    tgt = card.Target(shape, 160, pool_fill=0)
    _pack(tgt, shape, "normal", 7)
    before = _run(tgt, 1, 8, 41)
    d, f = shape.d_model, shape.d_ffn
    rows, cols = {"wq": (shape.q_dim, d), "wu": (f, d), "wd": (d, f), "lm_head": (shape.vocab, d)}[name]
    new = _weights("normal", rows, cols, 999)
    tgt.cfg.coded = 0
    tgt.pack(name, layer, new)
    tgt.cfg.coded = 1
    assert _refused(tgt)
    tgt.pack("wk", 0, _weights("normal", shape.kv_dim, d, 8))
    assert _refused(tgt)
    tgt.pack(name, layer, new)
    now, whole = _run(tgt, 1, 8, 41), _run(tgt, 0, 8, 41)
    assert all(torch.equal(a, b) for a, b in zip(now, whole)) and not torch.equal(now[0], before[0])


def test_a_target_takes_the_packed_weights_of_another():
    """... whichever of the two keeps the copy."""
    import paper_2508_04462_amd as card

    shape = SHAPES["odd"]
    tgts = {coded: card.Target(shape, 160, pool_fill=0, coded=coded) for coded in (False, True)}
    for tgt in tgts.values():
        _pack(tgt, shape, "outliers", 31)
    want = _run(tgts[False], 0, 8, 41)
    for coded in (False, True):
        tgt = card.Target(shape, 160, pool_fill=0, coded=coded)
        for blob in (tgts[True].packed, tgts[False].packed, tgts[True].packed):
            tgt.packed = blob
            assert all(torch.equal(a, b) for a, b in zip(_run(tgt, tgt.cfg.coded, 8, 41), want)), coded
        assert tgt.cfg.coded == 0  # once given a blob without a copy


@pytest.mark.parametrize("name,layers", [("llama8b", 2), ("qwen7b", 2), ("llama70b", 1)])
def test_wide_models_give_the_same_bits_on_either_kind_of_weights(name, layers):
    import paper_2508_04462_amd as card

    shape = ci.SHAPES[name].with_layers(layers)
    tgt = card.Target(shape, 160, pool_fill=0, coded=True)
    _pack(tgt, shape, "outliers", 41)
    for r in (1, 8, 13, 32):
        for got, want in zip(_run(tgt, 1, r, 41), _run(tgt, 0, r, 41)):
            assert torch.equal(got, want), (name, r)


def _sizes(max_ctx):
    """Bytes of a Target of the small shape with the copy: packed weights; workspace and page pools."""
    import paper_2508_04462_amd as card

    cfg = card.make_cfg(SHAPES["wide"], max_ctx)
    cfg.coded = 1
    return card.card_packed_weight_bytes(cfg), card.card_workspace_bytes(cfg) + 2 * card.card_kv_pool_bytes(cfg, max_ctx // 16)


def test_the_copy_needs_room_beside_everything_that_the_target_takes(monkeypatch):
    import paper_2508_04462_amd as card
    from paper_2508_04462_amd import runtime

    monkeypatch.setattr(runtime, "CODED_MIN_LAYER_BYTES", 0)
    monkeypatch.setattr(torch.cuda, "memory_reserved", lambda *a: 0)
    monkeypatch.setattr(torch.cuda, "memory_allocated", lambda *a: 0)
    both, rest = _sizes(160)
    total = 1 << 36
    for free, coded in ((total // 2 + both + rest, 1), (total // 2 + both + rest - 1, 0), (total // 2 + both, 0)):
        monkeypatch.setattr(torch.cuda, "mem_get_info", lambda *a: (free, total))
        tgt = card.Target(SHAPES["wide"], 160)
        assert tgt.cfg.coded == coded
        assert tgt.packed.numel() == card.card_packed_weight_bytes(tgt.cfg)


@pytest.mark.parametrize("nth", [0, 1, 2, 3])
def test_where_memory_runs_out_the_target_does_without_the_copy(monkeypatch, nth):
    import paper_2508_04462_amd as card
    from paper_2508_04462_amd import runtime

    monkeypatch.setattr(runtime, "CODED_MIN_LAYER_BYTES", 0)
    both, _ = _sizes(160)
    empty, taken = torch.empty, []

    def short(*a, **kw):
        if len(taken) <= nth and kw.get("dtype") == torch.uint8:
            taken.append(a[0])
            if len(taken) > nth:
                raise torch.cuda.OutOfMemoryError("out of memory")
        return empty(*a, **kw)

    monkeypatch.setattr(torch, "empty", short)
    tgt = card.Target(SHAPES["wide"], 160)
    assert taken[0] == both and len(taken) == nth + 1
    assert tgt.cfg.coded == 0 and tgt.packed.numel() == card.card_packed_weight_bytes(tgt.cfg) < both
    # asked for, it is taken or refused; not wanted, it is left out
    assert card.Target(SHAPES["wide"], 160, coded=True).cfg.coded == 1 and card.Target(SHAPES["wide"], 160, coded=False).cfg.coded == 0
    taken.clear()
    with pytest.raises(torch.cuda.OutOfMemoryError):
        card.Target(SHAPES["wide"], 160, coded=True)


@pytest.mark.parametrize("background", ["zeros", "normal"])
def test_every_bit_pattern_keeps_its_value(background):
    """A vocabulary head with one row per pattern of sixteen bits, among zeros (its bits are then all that a logit has) or ordinary weights."""
    import paper_2508_04462_amd as card

    shape = ci.ModelShape("patterns", 1, 256, 4, 4, 64, 256, 65536, ctx=64, r=8)
    tgt = card.Target(shape, 64, pool_fill=0, coded=True)
    _pack(tgt, shape, "normal", 11)
    head = _weights("normal", shape.vocab, shape.d_model, 12) if background == "normal" else torch.zeros(shape.vocab, shape.d_model,
                                                                                                         dtype=torch.bfloat16, device="cuda")
    rows = torch.arange(65536, device="cuda")
    head.view(torch.int16)[rows, rows * 37 % shape.d_model] = torch.where(rows < 32768, rows, rows - 65536).to(torch.int16)
    tgt.pack("lm_head", 0, head)
    for r in (1, 8, 13, 32):
        got = []
        for coded in (1, 0):
            tgt.cfg.coded = coded
            got.append(tgt.verify(0, -1, list(range(1, r + 1)), want_logits=True)["logits"].view(torch.int32))
        assert torch.equal(got[0], got[1]), (background, r)
        values = got[0].view(torch.float32)
        # (NaN where the pattern is one, at the least; almost all others are finite)
        assert bool(values[:, 0x7F81:0x7FFF].isnan().all()) and float(values.isfinite().float().mean()) > 0.9


@pytest.mark.parametrize("name", ["odd", "wide"])
@pytest.mark.parametrize("n", [12, 20, 60])  # pieces of 8 rows, of up to 16, of up to 32
def test_pieces_of_a_level_give_the_same_bits(name, n):
    """Calls of a level side by side, on whole weights and on the coded copy (kernels of their own for each)."""
    import paper_2508_04462_amd as card

    shape = SHAPES[name]
    tgt = card.Target(shape, 192, grid_wgs=64, pool_fill=0, coded=True)
    _pack(tgt, shape, "outliers", 21)
    tgt.enable_lanes(2)
    toks = [(37 * i + 5) % shape.vocab for i in range(41 + n)]
    st, rows = card.card_tree_mask_level(None, [-1] * n, 41, 41, 32, (41 + n - 32 + 31) // 32)
    assert st == card.CARD_OK
    out = []
    for coded in (1, 0):
        tgt.cfg.coded = coded
        tgt.k_pages.zero_()
        tgt.v_pages.zero_()
        tgt.prefill(toks[:41], chunk=8)
        lv = tgt.draft_level_wide(41, toks[41:], [41] * n, 41, rows, 32, 5)
        out.append([x.contiguous().view(torch.uint8).cpu() for x in (lv["topk_tokens"], lv["topk_probs"], tgt.k_pages, tgt.v_pages)])
        assert bool((lv["topk_tokens"] >= 0).all())
    assert all(torch.equal(a, b) for a, b in zip(*out))
