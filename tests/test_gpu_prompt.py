"""The prompt pass (card_prompt) against the CPU oracle: K and V of every position, the token behind
the last one, and a verification step on top of the cache it leaves.

Bars as for the verify step: K and V within one bf16 step (2^-8 of the largest value; layers above
the first also carry the rounding of the caches below: 2^-7), logits within 2e-2 of the row maximum,
tokens equal where the oracle's two best are more than 0.05 apart."""
import gc

import numpy as np
import pytest
import torch

import card_inputs as ci
from gpu_common import GAP, logits_rel_err, make_pair
from oracle import card_oracle as co

pytestmark = pytest.mark.gpu
TINY = ci.SHAPES["tiny"]
# head_dim 128, G = 4; the FFN ends inside a k-step, the vocabulary inside a tile, three layers
MID = ci.ModelShape("mid", 3, 512, 8, 2, 128, 1048, 3001, ctx=200, r=8)
# G = 3: row tiles that do not divide the heads; one layer; a QKV product with more tiles than workgroups
WIDE = ci.ModelShape("wide", 1, 192, 24, 8, 128, 264, 515, ctx=64, r=4)


def _check_kv(tgt, kv, shape, n):
    for layer in range(shape.n_layers):
        k, v = tgt.kv_gather(layer, 0, n)
        for got, ref in ((k, kv.k[layer][:n]), (v, kv.v[layer][:n])):
            assert np.abs(got.numpy() - ref).max() <= (2.0 ** -8 if layer == 0 else 2.0 ** -7) * np.abs(ref).max(), layer


def _top(row):
    order = np.argsort(row)[::-1]
    return int(order[0]), float(row[order[0]] - row[order[1]])


# around the row tiles (16) and row blocks (64) of the product kernel, one row more than a verify call
# takes, more than one pass (1024 rows), and a last pass that is a remainder
@pytest.mark.parametrize("shape,n", [(TINY, 33), (TINY, 64), (TINY, 65), (MID, 47), (MID, 48), (MID, 49), (MID, 63), (MID, 129),
                                     (MID, 1040), (TINY, 2100), (WIDE, 50), (WIDE, 81)],
                         ids=lambda p: getattr(p, "name", p))
def test_prompt_against_the_oracle(shape, n):
    r = 4
    tgt, w = make_pair(shape, 7, max_ctx=n + r, gain_jitter=0.2, pool_fill=0xFF)
    toks = ci.uniform_tokens(7, "ctx_tokens", n, n + r, shape.vocab).tolist()
    kv = co.OracleKV.empty(shape, n + r + 15)
    co.prefill(shape, w, kv, toks[: n - 1], chunk=256)
    row = co.forward_rows(shape, w, kv, toks[n - 1: n], n - 1)[0]
    g0 = tgt.prefill(toks[:n])
    best, gap = _top(row)
    assert g0 == best or (gap <= GAP and g0 in np.argsort(row)[-2:])
    _check_kv(tgt, kv, shape, n)
    # slots behind the last token are cleared with the page they are in: a step on top is finite and right
    ref = co.verify(shape, w, kv, n, -1, toks[n:], keep_logits=True)
    res = tgt.verify(n, -1, toks[n:], want_logits=True)
    assert torch.isfinite(res["logits"]).all()
    assert logits_rel_err(res["logits"], ref.logits) <= 2e-2


def _prompt(tgt, toks, ctx_len, rows, next_token=True):
    import paper_2508_04462_amd as card

    ws = torch.full((card.card_prompt_workspace_bytes(tgt.cfg, rows),), 0xFF, dtype=torch.uint8, device=tgt.device)
    dev = torch.tensor(toks, dtype=torch.int32, device=tgt.device)
    out = torch.full((1,), -9, dtype=torch.int32, device=tgt.device)
    st = card.card_prompt(tgt.cfg, tgt.packed, tgt.kv(-1), ctx_len, dev, len(toks), ws, rows, tgt._stream(), out if next_token else None)
    torch.cuda.synchronize()
    return st, int(out.item())


@pytest.mark.parametrize("shape,parts,rows", [(MID, (160, 37), 64), (TINY, (16, 100), 1), (MID, (32, 1), 128), (TINY, (112, 300), 192)],
                         ids=["mid-passes", "tiny-one-row-of-workspace", "mid-one-token", "tiny-passes"])
def test_prompt_in_parts_and_passes(shape, parts, rows):
    """A second prompt on top of the first (ctx_len > 0), and a workspace with room for fewer rows
    than the prompt has (several passes); the workspace starts as bf16 NaN patterns."""
    n = sum(parts)
    tgt, w = make_pair(shape, 8, max_ctx=n + 16, gain_jitter=0.2, pool_fill=0xFF)
    toks = ci.uniform_tokens(8, "ctx_tokens", 0, n, shape.vocab).tolist()
    kv = co.OracleKV.empty(shape, n + 16)
    co.prefill(shape, w, kv, toks[: n - 1], chunk=256)
    row = co.forward_rows(shape, w, kv, toks[n - 1:], n - 1)[0]
    assert _prompt(tgt, toks[: parts[0]], 0, rows, next_token=False) == (0, -9)
    st, token = _prompt(tgt, toks[parts[0]:], parts[0], rows)
    assert st == 0
    best, gap = _top(row)
    assert token == best or (gap <= GAP and token in np.argsort(row)[-2:])
    _check_kv(tgt, kv, shape, n)


def test_prompt_workspace_at_the_alignment_it_asks_for():
    import paper_2508_04462_amd as card

    tgt, _ = make_pair(MID, 6, max_ctx=112)
    toks = ci.uniform_tokens(6, "ctx_tokens", 0, 100, MID.vocab).tolist()
    want = tgt.prefill(toks)
    kv = [tgt.kv_gather(layer, 0, 100) for layer in range(MID.n_layers)]
    size = card.card_prompt_workspace_bytes(tgt.cfg, 100)
    ws = torch.full((size + 1024,), 0xFF, dtype=torch.uint8, device=tgt.device)
    at = (16 - ws.data_ptr()) % 1024  # 16 bytes behind a multiple of 1024
    dev = torch.tensor(toks, dtype=torch.int32, device=tgt.device)
    out = torch.full((1,), -9, dtype=torch.int32, device=tgt.device)
    tgt.k_pages.fill_(0xFF)
    tgt.v_pages.fill_(0xFF)
    assert card.card_prompt(tgt.cfg, tgt.packed, tgt.kv(-1), 0, dev, 100, ws[at:], 100, tgt._stream(), out) == card.CARD_OK
    assert int(out.item()) == want
    assert (ws[size + at:] == 0xFF).all()
    for layer in range(MID.n_layers):
        for a, b in zip(kv[layer], tgt.kv_gather(layer, 0, 100)):
            assert torch.equal(a, b)


@pytest.mark.parametrize("n", [20, 33, 300])
def test_prefill_reports_like_a_step(n):
    """`out` behind a prompt, whichever way it went (20 tokens: verify calls): the next token and the slots of this
    prompt, not of what ran before it; failed where a token lies outside the vocabulary."""
    tgt, _ = make_pair(TINY, 4, max_ctx=320)
    toks = ci.uniform_tokens(4, "ctx_tokens", 0, n, TINY.vocab).tolist()
    tgt.verify(0, -1, toks[:3])
    g0 = tgt.prefill(toks)
    taken, token, first, count = tgt.out.tolist()
    if n > 32:
        assert (taken, token, first, count) == (n, g0, 0, n)
    assert taken >= 1 and first + count <= n
    assert tgt.prefill([TINY.vocab] + toks[1:]) == tgt.prefill([TINY.vocab - 1] + toks[1:])
    for bad in (-1, TINY.vocab):
        tgt.prefill(toks[:-1] + [bad])
        assert tgt.out.tolist()[:2] == [-1, -1] and tgt.out.tolist()[3] == 0
        assert 0 <= tgt.prefill(toks) == g0


def test_prompt_on_weights_not_packed_for_this_grid():
    """As a verification step reports them: a blob that was never packed, and one packed for another grid size."""
    import paper_2508_04462_amd as card
    from paper_2508_04462_amd.synthetic import load_synthetic_weights

    toks = ci.uniform_tokens(3, "ctx_tokens", 0, 40, TINY.vocab).tolist()
    tgt, other = card.Target(TINY, 96), card.Target(TINY, 96, grid_wgs=64)
    load_synthetic_weights(other, TINY, 3)
    want = _prompt(other, toks, 0, 64)
    assert want[0] == 0 and 0 <= want[1] < TINY.vocab
    for blob in (torch.zeros_like(tgt.packed), other.packed):
        tgt.packed.copy_(blob)
        assert _prompt(tgt, toks, 0, 64) == (0, -1)
        assert tgt.verify(0, -1, toks[:4])["accepted_len"] == -1
        with pytest.raises(card.CardError):
            tgt.prefill(toks)
    load_synthetic_weights(tgt, TINY, 3)
    assert _prompt(tgt, toks, 0, 64) == want and tgt.prefill(toks) == want[1]


def test_prompt_refuses_what_it_cannot_do():
    import paper_2508_04462_amd as card

    tgt, _ = make_pair(TINY, 1, max_ctx=96)
    toks = list(range(40))
    assert _prompt(tgt, toks, 8, 64)[0] == card.CARD_EINVAL  # not at a page
    assert _prompt(tgt, toks, 64, 64)[0] == card.CARD_ECAPACITY
    assert _prompt(tgt, toks, -16, 64)[0] == card.CARD_EINVAL
    assert card.card_prompt_workspace_bytes(tgt.cfg, 0) == 0
    assert card.card_prompt(tgt.cfg, tgt.packed, tgt.kv(-1), 0, tgt.cand, 0, tgt.workspace, 64, None) == card.CARD_EINVAL
    with pytest.raises(card.CardError) as e:  # through the wrapper: as before
        tgt.prefill(list(range(100)))
    assert e.value.status == card.CARD_ECAPACITY
    # tokens outside the vocabulary are clamped, as the verify step's forward does
    assert tgt.prefill([5000, -3] + toks[2:]) == tgt.prefill([TINY.vocab - 1, 0] + toks[2:])


def test_prompt_workspace_can_be_given_back():
    tgt, _ = make_pair(MID, 5, max_ctx=200)
    toks = ci.uniform_tokens(5, "ctx_tokens", 0, 150, MID.vocab).tolist()
    gc.collect()  # (a model of an earlier test that is freed meanwhile would count)
    before = torch.cuda.memory_allocated()
    g0 = tgt.prefill(toks)
    assert torch.cuda.memory_allocated() > before
    tgt.release_prompt_workspace()
    assert torch.cuda.memory_allocated() == before
    assert tgt.prefill(toks) == g0


def test_prompt_on_a_full_device_goes_through_verify_calls(monkeypatch):
    """Where the device has no room for the prompt's workspace a prompt is what it was without it:
    verify calls of 32 rows (the same bits), with room for fewer rows only, more passes."""
    from paper_2508_04462_amd import runtime

    tgt, w = make_pair(TINY, 4, max_ctx=320)
    toks = ci.uniform_tokens(4, "ctx_tokens", 0, 300, TINY.vocab).tolist()
    real = runtime.B.card_prompt_workspace_bytes
    monkeypatch.setattr(runtime, "PROMPT_MIN_TOKENS", 10 ** 9)
    g0 = tgt.prefill(toks)
    by_calls = tgt.kv_gather(1, 0, 300)
    monkeypatch.setattr(runtime, "PROMPT_MIN_TOKENS", 33)
    for most, rows in ((0, 0), (80, 75)):  # (asked for 300, then 150, then 75 rows)
        monkeypatch.setattr(runtime.B, "card_prompt_workspace_bytes", lambda cfg, n: real(cfg, n) if n <= most else 1 << 45)
        tgt._prompt_ws, tgt._prompt_rows = None, 0
        got = tgt.prefill(toks)
        assert tgt._prompt_rows == rows
        k, v = tgt.kv_gather(1, 0, 300)
        if rows == 0:
            assert got == g0 and torch.equal(k, by_calls[0]) and torch.equal(v, by_calls[1])
        else:
            assert (k - by_calls[0]).abs().max() <= 2.0 ** -7 * by_calls[0].abs().max()
