"""Steps of models that are too small for the whole grid: workgroups that would have neither a tile nor an attention task are not
launched.  Nothing else may depend on that: neither the packed weights nor a result."""
import dataclasses

import pytest
import torch

import card_inputs as ci

pytestmark = pytest.mark.gpu

TINY = ci.SHAPES["tiny"]  # gate/up: 86 tiles, the widest
MID = ci.ModelShape("mid", 3, 512, 8, 2, 128, 1048, 3001, ctx=200, r=8)  # vocabulary: 188 tiles


def _target(shape, max_ctx, **kw):
    import paper_2508_04462_amd as card
    from paper_2508_04462_amd.synthetic import load_synthetic_weights

    tgt = card.Target(shape, max_ctx, pool_fill=0, **kw)
    load_synthetic_weights(tgt, shape, 3, 0.2)
    return tgt


def _tokens(shape, n):
    return ci.uniform_tokens(3, "ctx_tokens", 0, n, shape.vocab).tolist()


def test_packed_weights_serve_every_context_size_and_every_equal_configuration():
    """One blob, two default models of other context sizes, and a configuration that the caller builds."""
    import paper_2508_04462_amd as card
    from paper_2508_04462_amd.runtime import make_cfg

    toks = _tokens(TINY, 45)
    short, long = _target(TINY, 128), card.Target(TINY, 4096, pool_fill=0)
    long.packed.copy_(short.packed)
    for tgt in (short, long):
        tgt.prefill(toks[:40])
    a, b = (t.verify(40, -1, toks[40:], want_logits=True) for t in (short, long))
    assert a["accepted_len"] >= 0 and b["accepted_len"] >= 0
    assert torch.equal(a["logits"], b["logits"])
    cfg = make_cfg(TINY, 128)
    assert bytes(cfg) == bytes(short.cfg)
    short.out.fill_(-7)
    assert card.card_verify(cfg, short.packed, short.kv(-1), 40, short.cand, 5, short.workspace, short._stream(), short.out,
                            short.row_argmax) == card.CARD_OK
    torch.cuda.synchronize()
    assert short.out[0].item() == a["accepted_len"] and short.row_argmax[:5].tolist() == a["row_argmax"]


# Grids of fewer positions than the widest matrix has tiles, of as many, of more, with and without positions left over.  (Above eight
# rows multiples of eight only: other grids sum the down-projection in another order.)
@pytest.mark.parametrize("shape,r,grids", [
    (TINY, 1, (85, 86, 88, 96, 256)), (TINY, 8, (85, 87, 88, 104, 256)), (TINY, 13, (80, 88, 96, 256)), (TINY, 32, (80, 88, 256)),
    (dataclasses.replace(TINY, name="tiny-v1395", vocab=1395), 8, (87, 88, 256)),  # 88 tiles
    (dataclasses.replace(TINY, name="tiny-v1409", vocab=1409), 8, (88, 96, 256)),  # 89
    (MID, 5, (131, 188, 192, 208, 256)), (MID, 16, (128, 192, 200, 256)), (MID, 20, (184, 192, 256))],
    ids=lambda v: v.name if hasattr(v, "name") else None)
def test_a_result_does_not_depend_on_how_many_workgroups_have_work(shape, r, grids):
    """Bit for bit."""
    toks = _tokens(shape, 31 + r)
    out = []
    for grid in grids:
        tgt = _target(shape, 128, grid_wgs=grid)
        tgt.prefill(toks[:31], chunk=8)
        res = tgt.verify(31, -1, toks[31:], want_logits=True)
        assert res["accepted_len"] >= 0
        out.append((res["logits"], *tgt.kv_gather(shape.n_layers - 1, 0, 31 + r)))
    for other in out[1:]:
        for x, y in zip(out[0], other):
            assert torch.equal(x, y)


def test_workgroups_that_were_left_out_come_back():
    """A short call leaves workgroups out that a long one (256 attention tasks) needs, on one workspace.  The barrier flags of those left out
    keep up with the calls: far enough behind, one would look ahead of the call that waits for it."""
    ctx = 8160
    tgt, fresh = _target(TINY, 8192), _target(TINY, 8192)
    toks = _tokens(TINY, 32)
    short = [t.verify(0, -1, toks[:8], want_logits=True)["logits"] for t in (tgt, fresh)]
    assert torch.equal(*short)
    want = fresh.verify(ctx, -1, toks, want_logits=True)["logits"]
    assert torch.equal(tgt.verify(ctx, -1, toks, want_logits=True)["logits"], want)
    # 32 copies of 256 flags, all of them at the call's last barrier
    words = tgt.workspace.view(torch.int32).clone()
    start = next(i for i in range(0, words.numel() - 8191, 64)
                 if words[i] != 0 and words[i + 8191] == words[i] and bool((words[i:i + 8192] == words[i]).all()))
    last = int(words[start])
    assert torch.equal(tgt.verify(0, -1, toks[:8], want_logits=True)["logits"], short[0])
    flags = tgt.workspace.view(torch.int32)[start:start + 8192].view(32, 256)
    assert (flags > last).all() and (flags[:, 255] < flags[:, 0]).all()
    assert torch.equal(tgt.verify(ctx, -1, toks, want_logits=True)["logits"], want)
