"""Draft-side cache construction on the device against the CPU oracle (Cache Construction,
eqs. (1)-(9); Mask Construction for Draft Model): card_draft_level (tree forward with the
ancestor mask, fused per-row top-k and probabilities) and card_cache_select (path scores and the
global top-K), through the C ABI.

Bars: logits within 2e-2 of the row maximum (as for the verify step); log-probabilities of the
returned tokens within 5e-3 of the oracle's; the returned token SET equals the oracle's top-k
wherever the k-th and (k+1)-th oracle logits are more than 0.05 apart, and the order of two
neighbours is checked wherever they are that far apart; selected tuples equal the oracle's
wherever the scores around the cut and between neighbours are decisive."""
import numpy as np
import pytest
import torch

import card_inputs as ci
from gpu_common import logits_rel_err, make_pair
from oracle import card_oracle as co
from oracle.cache_oracle import build_level, tree_mask

pytestmark = pytest.mark.gpu
TINY = ci.SHAPES["tiny"]
MID = ci.ModelShape("mid", 3, 512, 8, 2, 128, 1048, 3001, ctx=200, r=8)
GAP = 0.05


def _check_topk(tk, tp, ref_logits, k):
    """tk, tp: device results of one row; ref_logits: the oracle's row."""
    order = sorted(range(ref_logits.shape[0]), key=lambda t: (-ref_logits[t], t))
    lse = np.log(np.exp(ref_logits - ref_logits.max()).sum()) + ref_logits.max()
    toks = tk.tolist()
    assert len(set(toks)) == k and all(0 <= t < ref_logits.shape[0] for t in toks)
    for j, t in enumerate(toks):  # probabilities of whatever was returned
        assert abs(np.log(tp[j]) - (ref_logits[t] - lse)) <= 5e-3, (j, t)
    if ref_logits[order[k - 1]] - ref_logits[order[k]] > GAP:
        assert set(toks) == set(order[:k])
    n_ord = 0
    for j in range(k - 1):
        assert tp[j] >= tp[j + 1]
        if ref_logits[order[j]] - ref_logits[order[j + 1]] > GAP and all(
                abs(ref_logits[order[i]] - ref_logits[order[i + 1]]) > GAP for i in range(max(0, j - 1), min(k, j + 2))):
            n_ord += int(toks[j] == order[j])
    return n_ord


def _levels(rng, widths, vocab):
    out, prev = [], 0
    for l, n in enumerate(widths):
        toks = rng.integers(0, vocab, size=n).tolist()
        parents = [-1] * n if l == 0 else rng.integers(0, prev, size=n).tolist()
        out.append((toks, parents))
        prev = n
    return out


@pytest.mark.parametrize("shape,ctx_len,widths,k", [(TINY, 37, [3, 5, 4, 6], 4), (MID, 61, [2, 8, 17, 32], 10),
                                                    (MID, 16, [40], 16), (TINY, 100, [9, 33, 12], 7)],
                         ids=["tiny", "mid", "mid-wide-level", "tiny-wide"])
def test_draft_level_against_the_oracle(shape, ctx_len, widths, k):
    tgt, w = make_pair(shape, 9, max_ctx=320, gain_jitter=0.2)
    rng = np.random.default_rng(9)
    ctx = ci.uniform_tokens(9, "ctx_tokens", 0, ctx_len, shape.vocab).tolist()
    kv = co.OracleKV.empty(shape, 320)
    co.prefill(shape, w, kv, ctx)
    tgt.prefill(ctx, chunk=29)
    levels = _levels(rng, widths, shape.vocab)
    ref_mask = tree_mask([p for _, p in levels])
    offs = np.cumsum([0] + widths)
    mask_base, tree_base = ctx_len // 16 * 16, (ctx_len + 15) // 16 * 16
    words = (tree_base + int(offs[-1]) - mask_base + 31) // 32
    import paper_2508_04462_amd as card

    prev_rows, n_ord = None, 0
    for l, (toks, parents) in enumerate(levels):
        n = len(toks)
        first = tree_base + int(offs[l])
        st, rows = card.card_tree_mask_level(prev_rows, parents, first, ctx_len, mask_base, words)
        assert st == card.CARD_OK
        visible = [list(range(ctx_len)) + [tree_base + int(j) for j in np.flatnonzero(ref_mask[offs[l] + i])] for i in range(n)]
        ref = co.forward_tree_rows(shape, w, kv, toks, [ctx_len + l] * n, [first + i for i in range(n)], visible)
        for c0 in range(0, n, 32):  # a level wider than 32 rows takes several calls
            c1 = min(n, c0 + 32)
            res = tgt.draft_level(ctx_len, toks[c0:c1], [ctx_len + l] * (c1 - c0), first + c0, rows[c0:c1], mask_base, k,
                                  want_logits=True)
            assert logits_rel_err(res["logits"], ref[c0:c1]) <= 2e-2
            tk, tp = res["topk_tokens"].cpu().numpy(), res["topk_probs"].cpu().double().numpy()
            for i in range(c0, c1):
                n_ord += _check_topk(tk[i - c0], tp[i - c0], ref[i], k)
        prev_rows = rows
        # the keys the level wrote are the oracle's (last layer, first rows)
        kk, vv = tgt.kv_gather(shape.n_layers - 1, first, min(n, 8))
        ref_k = kv.k[-1][first: first + min(n, 8)]
        assert np.abs(kk.numpy() - ref_k).max() <= 2.0 ** -7 * np.abs(ref_k).max()
    assert n_ord > 0


def test_select_exact_on_dyadic_scores_with_ties():
    """eqs. (3)-(7) on inputs whose products are exact in fp32: the result must equal the oracle's
    tuple for tuple, ties included (equal scores in parent, then rank order)."""
    import paper_2508_04462_amd as card

    rng = np.random.default_rng(1)
    for M, k, K in [(5, 4, 7), (50, 10, 50), (100, 16, 100), (3, 2, 10)]:
        vocab = 64
        probs = np.zeros((M, vocab))
        toks = np.zeros((M, k), dtype=np.int32)
        pv = np.zeros((M, k), dtype=np.float32)
        for i in range(M):
            vals = np.sort(rng.integers(1, 16, size=k))[::-1] / 64.0  # few distinct values: many ties
            ids = np.sort(rng.choice(vocab, size=k, replace=False))
            # descending probability, ascending token among equals: what eq. (2) hands over
            order = sorted(range(k), key=lambda j: (-vals[j], ids[j]))
            toks[i], pv[i] = ids[order], vals[order]
            probs[i, ids] = vals
        sigma = (rng.integers(1, 8, size=M) / 8.0).astype(np.float32)
        rt, rs, rp = build_level(probs, sigma.astype(np.float64), K, k)
        dev = "cuda:0"
        ot = torch.empty(K, dtype=torch.int32, device=dev)
        os_ = torch.empty(K, dtype=torch.float32, device=dev)
        op = torch.empty(K, dtype=torch.int32, device=dev)
        n = card.card_cache_select(torch.from_numpy(sigma).to(dev), torch.from_numpy(toks).to(dev),
                                   torch.from_numpy(pv).to(dev), M, k, K, ot, os_, op)
        torch.cuda.synchronize()
        assert n == min(K, M * k) == len(rt)
        assert ot[:n].tolist() == rt.tolist() and op[:n].tolist() == rp.tolist()
        np.testing.assert_array_equal(os_[:n].cpu().numpy().astype(np.float64), rs)
    # parents switched off by a negative token take no part; outputs behind the last tuple are marked empty
    M, k, K, dev = 6, 3, 8, "cuda:0"
    toks = torch.arange(M * k, dtype=torch.int32, device=dev).reshape(M, k)
    toks[[0, 1, 3, 5]] = -1
    pv = torch.tensor([[0.5, 0.25, 0.125]] * M, dtype=torch.float32, device=dev)
    sigma = torch.tensor([1.0, 1.0, 0.5, 1.0, 1.0, 1.0], dtype=torch.float32, device=dev)
    ot = torch.empty(K, dtype=torch.int32, device=dev)
    os_ = torch.empty(K, dtype=torch.float32, device=dev)
    op = torch.empty(K, dtype=torch.int32, device=dev)
    assert card.card_cache_select(sigma, toks, pv, M, k, K, ot, os_, op) == K
    torch.cuda.synchronize()
    # equal scores: the lower parent index first
    assert ot.tolist() == [12, 6, 13, 7, 14, 8, -1, -1] and op.tolist() == [4, 2, 4, 2, 4, 2, -1, -1]
    assert os_.tolist() == [0.5, 0.25, 0.25, 0.125, 0.125, 0.0625, 0.0, 0.0]
    bad = torch.zeros(4, dtype=torch.int32, device="cuda:0")
    assert card.card_cache_select(bad, bad, bad, 200, 16, 10, bad, bad, bad) == card.CARD_ERANGE


@pytest.mark.parametrize("M,k,K", [(1, 1, 1), (16, 4, 64), (13, 5, 65), (21, 3, 40), (16, 8, 128), (43, 3, 129), (128, 16, 2048), (127, 16, 100)])
def test_select_at_the_edges_of_its_workgroups(M, k, K):
    """Keys are sorted as a power of two of them, 128 per wavefront: counts around 64 and 128, the largest
    (2048), odd ones, a third of the tuples empty, many equal scores."""
    import paper_2508_04462_amd as card

    rng = np.random.default_rng(M * 100 + k)
    toks = rng.integers(0, 1000, size=(M, k)).astype(np.int32)
    toks[rng.random((M, k)) < 0.33] = -1
    prob = (rng.integers(0, 8, size=(M, k)) / 8.0).astype(np.float32)  # (a score of zero is a score)
    sigma = (rng.integers(1, 5, size=M) / 4.0).astype(np.float32)
    score = (prob * sigma[:, None]).reshape(-1)
    order = [i for i in sorted(range(M * k), key=lambda i: (-score[i], i)) if toks.reshape(-1)[i] >= 0]
    n = min(K, M * k)
    want = order[:n]
    dev = "cuda:0"
    ot = torch.full((n,), -7, dtype=torch.int32, device=dev)
    os_, op = torch.full((n,), -7.0, dtype=torch.float32, device=dev), torch.full((n,), -7, dtype=torch.int32, device=dev)
    assert card.card_cache_select(torch.from_numpy(sigma).to(dev), torch.from_numpy(toks).to(dev), torch.from_numpy(prob).to(dev), M, k,
                                  K, ot, os_, op) == n
    torch.cuda.synchronize()
    pad = n - len(want)
    assert ot.tolist() == toks.reshape(-1)[want].tolist() + [-1] * pad
    assert os_.tolist() == score[want].tolist() + [0.0] * pad
    assert op.tolist() == [i // k for i in want] + [-1] * pad


@pytest.mark.parametrize("M,k,K", [(100, 8, 100), (128, 16, 2048), (70, 5, 33)])
@pytest.mark.parametrize("over", ["sigma", "probs", "tokens", "inside"])
def test_select_in_place(M, k, K, over):
    """An output over an input, or over a part of one: the same as with arrays of its own."""
    import paper_2508_04462_amd as card

    g = torch.Generator().manual_seed(M)
    n = min(K, M * k)
    toks = torch.randint(-1, 1000, (M, k), generator=g, dtype=torch.int32).cuda()
    prob, sigma = torch.rand((M, k), generator=g).cuda(), torch.rand(max(M, n), generator=g).cuda()
    own = [torch.full((n,), -7, dtype=t, device="cuda") for t in (torch.int32, torch.float32, torch.int32)]
    assert card.card_cache_select(sigma, toks, prob, M, k, K, *own) == n
    want = [t.clone() for t in own]
    outs = list(own)
    if over == "tokens":
        outs[0] = toks.view(-1)[:n]
    else:
        outs[1] = {"sigma": sigma[:n], "probs": prob.view(-1)[:n], "inside": prob.view(-1)[M * k - n:]}[over]
    assert card.card_cache_select(sigma, toks, prob, M, k, K, *outs) == n
    torch.cuda.synchronize()
    for a, b in zip(outs, want):
        assert torch.equal(a, b)


def test_three_levels_built_on_the_device_and_written_to_the_cache():
    """Cache construction end to end: level after level, the device expands the current nodes
    (card_draft_level), scores and selects the next level (card_cache_select), the host stores it
    (card_cache_write) and derives the next mask rows; the oracle does the same from its own
    distributions.  Levels are compared while every choice up to them is decisive."""
    import paper_2508_04462_amd as card

    shape, ctx_len, K, k, depth = MID, 45, 12, 5, 3
    tgt, w = make_pair(shape, 4, max_ctx=320, gain_jitter=0.2)
    ctx = ci.uniform_tokens(4, "ctx_tokens", 0, ctx_len, shape.vocab).tolist()
    kv = co.OracleKV.empty(shape, 320)
    g0 = co.prefill(shape, w, kv, ctx)
    assert tgt.prefill(ctx) == g0
    mask_base, tree_base = ctx_len // 16 * 16, (ctx_len + 15) // 16 * 16
    words = (tree_base + 1 + K * depth - mask_base + 31) // 32
    cache = card.CandidateCache(K=K, max_depth=depth + 1)
    cache.write(0, [g0], [-1], [1.0])
    # oracle state
    o_toks, o_par, o_sig, o_vis = [g0], [-1], np.array([1.0]), [list(range(ctx_len)) + [tree_base]]
    # device state
    d_toks, d_par, d_sig = [g0], [-1], torch.ones(1, dtype=torch.float32, device="cuda:0")
    st, d_rows = card.card_tree_mask_level(None, [-1], tree_base, ctx_len, mask_base, words)
    first, compared = tree_base, 0
    for l in range(depth):
        n = len(o_toks)
        ref = co.forward_tree_rows(shape, w, kv, o_toks, [ctx_len + l] * n, [first + i for i in range(n)], o_vis)
        probs = co.softmax_rows(ref)
        rt, rs, rp = build_level(probs, o_sig, K, k)
        same_inputs = d_toks == o_toks and d_par == o_par
        res = tgt.draft_level(ctx_len, d_toks, [ctx_len + l] * len(d_toks), first, d_rows, mask_base, k)
        ot = torch.empty(K, dtype=torch.int32, device="cuda:0")
        os_ = torch.empty(K, dtype=torch.float32, device="cuda:0")
        op = torch.empty(K, dtype=torch.int32, device="cuda:0")
        cnt = card.card_cache_select(d_sig, res["topk_tokens"], res["topk_probs"], len(d_toks), k, K, ot, os_, op)
        torch.cuda.synchronize()
        assert cnt == min(K, len(d_toks) * k)
        nt, ns, npar = ot[:cnt].tolist(), os_[:cnt].cpu().numpy().astype(np.float64), op[:cnt].tolist()
        assert cache.write(l + 1, nt, npar, ns.tolist()) == card.CARD_OK
        # decisive: every oracle score differs from its neighbours (and from the first one cut) by > 2 %
        pool = sorted((float(probs[i, t]) * float(o_sig[i]) for i in range(n) for t in np.argsort(-probs[i])[:k]), reverse=True)
        cut = pool[: len(rt) + 1]
        decisive = all(cut[j] > 1.02 * cut[j + 1] for j in range(len(cut) - 1))
        if same_inputs and decisive:
            assert nt == rt.tolist() and npar == rp.tolist()
            np.testing.assert_allclose(ns, rs, rtol=5e-3)
            compared += 1
        # next level: oracle
        new_first = first + n
        o_vis = [o_vis[p] + [new_first + i] for i, p in enumerate(rp.tolist())]
        o_toks, o_par, o_sig = rt.tolist(), rp.tolist(), rs
        # next level: device (mask rows from the host helper, scores stay on the device)
        st, d_rows = card.card_tree_mask_level(d_rows, npar, new_first, ctx_len, mask_base, words)
        assert st == card.CARD_OK
        d_toks, d_par, d_sig = nt, npar, os_[:cnt].clone()
        first = new_first
    assert compared >= 1
    assert cache.depth() == depth + 1
    hit, path, score = cache.query(g0, depth + 1)
    assert hit and path[0] == g0 and len(path) == depth + 1


def test_a_wide_level_in_calls_side_by_side_equals_the_calls_one_after_the_other():
    """A level of 100 nodes on four lanes (each call on its own 64 workgroups, workspace and
    stream) gives bit for bit what four calls in a row on the same grid give, and leaves the same
    keys in the cache."""
    import paper_2508_04462_amd as card
    from paper_2508_04462_amd.synthetic import load_synthetic_weights

    shape, seed, ctx_len, n, k = MID, 21, 70, 100, 8
    tgt = card.Target(shape, 320, max_r=32, grid_wgs=64)
    load_synthetic_weights(tgt, shape, seed, 0.2)
    tgt.enable_lanes(4)
    tgt._level_ws = None  # (no room for the one-pass route's workspace)
    ctx = ci.uniform_tokens(seed, "ctx_tokens", 0, ctx_len, shape.vocab).tolist()
    tgt.prefill(ctx)
    rng = np.random.default_rng(seed)
    mask_base, first = ctx_len // 16 * 16, 80
    words = (first + 1 + 2 * n - mask_base + 31) // 32
    st, root_row = card.card_tree_mask_level(None, [-1], first, ctx_len, mask_base, words)
    tgt.draft_level(ctx_len, [5], [ctx_len], first, root_row, mask_base, k)
    toks = rng.integers(0, shape.vocab, size=n).tolist()
    out = {}
    for name, base in (("row", first + 1), ("wide", first + 1)):  # the same slots: the same sums in the same order
        st, rows = card.card_tree_mask_level(root_row, [0] * n, base, ctx_len, mask_base, words)
        assert st == card.CARD_OK
        if name == "wide":
            res = tgt.draft_level_wide(ctx_len, toks, [ctx_len + 1] * n, base, rows, mask_base, k)
            tk, tp = res["topk_tokens"].cpu(), res["topk_probs"].cpu()
        else:
            parts = [tgt.draft_level(ctx_len, toks[c:c + 32], [ctx_len + 1] * len(toks[c:c + 32]), base + c, rows[c:c + 32],
                                     mask_base, k) for c in range(0, n, 32)]
            tk = torch.cat([p["topk_tokens"].cpu() for p in parts])
            tp = torch.cat([p["topk_probs"].cpu() for p in parts])
        kk, vv = tgt.kv_gather(shape.n_layers - 1, base, n)
        out[name] = (tk, tp, kk, vv)
    for a, b in zip(out["row"], out["wide"]):
        assert torch.equal(a, b)
    assert (out["wide"][0] >= 0).all()


def _level_twice(shape, seed, ctx_len, first, n, k, lanes, grid=64, per=None):
    """Roots from the last page in use on, and a level of n nodes behind them from slot `first`, on two models with the same weights whose pools
    start as 0xFF bytes (NaN patterns): forwarded in a row on the first, in calls of `per` rows or as `lanes` lanes would cut it; -> both
    models, the row call's results, and the level's arguments."""
    import paper_2508_04462_amd as card
    from paper_2508_04462_amd.runtime import level_pieces
    from paper_2508_04462_amd.synthetic import load_synthetic_weights

    ctx = ci.uniform_tokens(seed, "ctx_tokens", 0, ctx_len, shape.vocab).tolist()
    mask_base, base = ctx_len // 16 * 16, first - ((first - 1) % 16 + 1)
    words = (first + n - mask_base + 31) // 32
    base, roots = max(base, ctx_len), first - max(base, ctx_len)
    st, root_rows = card.card_tree_mask_level(None, [-1] * roots, base, ctx_len, mask_base, words)
    assert st == card.CARD_OK
    st, rows = card.card_tree_mask_level(root_rows, [i % roots for i in range(n)], first, ctx_len, mask_base, words)
    assert st == card.CARD_OK
    tgts = []
    for _ in range(2):
        tgt = card.Target(shape, 320, max_r=32, grid_wgs=grid, pool_fill=0xFF)
        if tgts:
            tgt.packed.copy_(tgts[0].packed)
        else:
            load_synthetic_weights(tgt, shape, seed, 0.2)
        if lanes:
            tgt.enable_lanes(lanes)
        tgt.prefill(ctx)
        tgt.draft_level(ctx_len, list(range(5, 5 + roots)), [ctx_len] * roots, base, root_rows, mask_base, k)
        tgts.append(tgt)
    toks = ci.uniform_tokens(seed, "ctx_tokens", 1, n, shape.vocab).tolist()
    pieces = [(a, min(n, a + per)) for a in range(0, n, per)] if per else level_pieces(n, lanes)
    parts = [tgts[0].draft_level(ctx_len, toks[a:b], [ctx_len + 1] * (b - a), first + a, rows[a:b], mask_base, k) for a, b in pieces]
    want = tuple(torch.cat([p[key].cpu() for p in parts]) for key in ("topk_tokens", "topk_probs"))
    return tgts, want, toks, rows, mask_base, pieces


def _forward_level(route, tgt, blob, toks, rows, mask_base, first, n, k, per=None):
    """A level behind 70 tokens by the entry points themselves, one call after the other."""
    import paper_2508_04462_amd as card
    from paper_2508_04462_amd.runtime import level_pieces

    dev, words = tgt.device, len(rows[0])
    tok = torch.tensor(toks, dtype=torch.int32, device=dev)
    pos = torch.full((n,), 71, dtype=torch.int32, device=dev)
    mask = torch.tensor([[w - (1 << 32) if w >= 1 << 31 else w for w in row] for row in rows], dtype=torch.int32, device=dev)
    tk = torch.full((n, k), -7, dtype=torch.int32, device=dev)
    tp = torch.full((n, k), -7.0, dtype=torch.float32, device=dev)
    args = lambda a: card.CardTreeRows(tok[a:].data_ptr(), pos[a:].data_ptr(), first + a, mask[a:].data_ptr(), words, mask_base)  # noqa: E731
    pieces = level_pieces(n, 2)
    if route == "one pass":
        ws = torch.empty(card.card_level_workspace_bytes(tgt.cfg), dtype=torch.uint8, device=dev).fill_(0xFF)
        assert card.card_draft_level_wide(tgt.cfg, blob, tgt.kv(-1), 70, args(0), n, per or max(16, pieces[0][1]), k, ws, tgt._stream(),
                                          tk, tp) == card.CARD_OK
    elif route == "call":
        assert card.card_draft_level(tgt.cfg, blob, tgt.kv(-1), 70, args(0), n, k, tgt.workspace, tgt._stream(), tk, tp,
                                     None) == card.CARD_OK
    else:
        for a, b in pieces:
            assert card.card_draft_level_piece(tgt.cfg, blob, tgt.kv(-1), 70, args(a), b - a, first, first + n, k, tgt.workspace,
                                               tgt._stream(), tk[a:b], tp[a:b], None) == card.CARD_OK
    torch.cuda.synchronize()
    return tk.cpu(), tp.cpu()


def _same_level(tgts, want, got, shape, first, n):
    assert torch.equal(want[0], got[0]) and torch.equal(want[1], got[1])
    end = (first + n + 15) // 16 * 16
    for layer in range(shape.n_layers):
        for one, two in zip(tgts[0].kv_gather(layer, 0, first + n), tgts[1].kv_gather(layer, 0, first + n)):
            assert torch.equal(one.view(torch.int32), two.view(torch.int32))  # (slots that nobody wrote hold NaN)
        assert torch.isfinite(tgts[1].kv_gather(layer, first, n)[1]).all()
        if end > first + n and end - 16 >= first:  # a page that the level opened: cleared behind the level
            assert (tgts[1].kv_gather(layer, first + n, end - first - n)[1] == 0).all()


# levels that start and end anywhere in a page; cuts inside pages
LEVELS = [(80, 33), (81, 40), (87, 48), (95, 17), (79, 12), (81, 100), (80, 100), (93, 66), (88, 9)]


@pytest.mark.parametrize("first,n", LEVELS)
@pytest.mark.parametrize("shape", [TINY, MID], ids=["tiny", "mid"])
def test_pieces_of_a_level_in_any_order(shape, first, n):
    """The last piece first: a piece that opens a page leaves the slots of the level's other pieces alone, and a
    piece that runs before its neighbours does not mind what their slots hold."""
    import paper_2508_04462_amd as card

    k = 6
    tgts, want, toks, rows, mask_base, pieces = _level_twice(shape, 23, 70, first, n, k, 2)
    tgt, dev = tgts[1], tgts[1].device
    tok = torch.tensor(toks, dtype=torch.int32, device=dev)
    pos = torch.full((n,), 71, dtype=torch.int32, device=dev)
    mask = torch.tensor([[w - (1 << 32) if w >= 1 << 31 else w for w in row] for row in rows], dtype=torch.int32, device=dev)
    tk = torch.full((n, k), -7, dtype=torch.int32, device=dev)
    tp = torch.zeros((n, k), dtype=torch.float32, device=dev)
    for a, b in reversed(pieces):
        r = card.CardTreeRows(tok[a:b].data_ptr(), pos[a:b].data_ptr(), first + a, mask[a:b].data_ptr(), len(rows[0]), mask_base)
        assert card.card_draft_level_piece(tgt.cfg, tgt.packed, tgt.kv(-1), 70, r, b - a, first, first + n, k, tgt.workspace,
                                           tgt._stream(), tk[a:b], tp[a:b]) == card.CARD_OK
    torch.cuda.synchronize()
    _same_level(tgts, want, (tk.cpu(), tp.cpu()), shape, first, n)


@pytest.mark.parametrize("lanes,one_pass", [(2, False), (4, False), (4, True)])
@pytest.mark.parametrize("first,n", LEVELS)
def test_a_wide_level_from_any_slot_leaves_what_calls_in_a_row_leave(first, n, lanes, one_pass):
    """Pieces side by side that share a page, and one pass (more than 32 rows), on pools that nobody has written these slots of before."""
    tgts, want, toks, rows, mask_base, _ = _level_twice(MID, 24, 70, first, n, 5, lanes)
    assert (tgts[1]._level_ws is not None) == (lanes == 4)
    if not one_pass:
        tgts[1]._level_ws = None
    res = tgts[1].draft_level_wide(70, toks, [71] * n, first, rows, mask_base, 5)
    _same_level(tgts, want, (res["topk_tokens"].cpu(), res["topk_probs"].cpu()), MID, first, n)


# several passes (24 and 16 rows per call, the last of eight and less), two row tiles of which the second has one row, one pass
# of exactly eight row tiles; the widest k
@pytest.mark.parametrize("shape,first,n,lanes,k", [(MID, 87, 200, 3, 16), (TINY, 80, 150, 4, 1), (MID, 81, 49, 2, 7), (MID, 80, 128, 2, 16),
                                                   (MID, 95, 33, 3, 5)])
def test_one_pass_over_a_wide_level_equals_its_calls(shape, first, n, lanes, k):
    tgts, want, toks, rows, mask_base, pieces = _level_twice(shape, 26, 70, first, n, k, lanes)
    got = _forward_level("one pass", tgts[1], tgts[1].packed, toks, rows, mask_base, first, n, k, pieces[0][1])
    _same_level(tgts, want, got, shape, first, n)


# Every tile choice of the pass's products, and vocabularies of many tiles per lane.  Weight tiles x row tiles per wavefront of QKV | O and
# down | gate/up | vocabulary:
WIDTHS = [
    ("llama1b", 2, 100, 32, 8, 128),   # 2x2 | 1x2 | 1x4 | 2x8, the last call of four rows
    ("llama1b", 1, 28, 24, 16, 48),    # 1x2 | 1x2 | 1x4 | 2x4, four rows; 41 tiles per lane: more columns than the top-k keeps in registers
    ("llama8b", 2, 100, 32, 8, 256),   # 1x2 | 2x2 | 2x4 | 2x8, four rows
    ("llama8b", 1, 60, 32, 3, 128),    # 2x2 | 1x2 | 1x4 | 2x4
    ("qwen7b", 2, 53, 24, 8, 128),     # 2x2 | 2x2 | 2x8 | 2x8, five rows
    ("qwen7b", 1, 32, 24, 1, 200),     # 2x2 | 1x2 | 2x4 | 2x4, eight rows
    ("llama70b", 1, 114, 32, 5, 256),  # 1x2 | 2x2 | 2x8 | 2x8, the last call of 18
    ("tiny", 2, 53, 24, 6, 256),       # 1x2 | 1x2 | 1x4 | 1x4; calls that leave out the workgroups without work
]


@pytest.mark.parametrize("model,layers,n,per,k,grid", WIDTHS, ids=[f"{w[0]}-{w[2]}" for w in WIDTHS])
def test_one_pass_over_a_wide_level_of_real_widths_equals_its_calls(model, layers, n, per, k, grid):
    shape, first = ci.SHAPES[model].with_layers(layers), 85
    tgts, want, toks, rows, mask_base, _ = _level_twice(shape, 29, 70, first, n, k, 0, grid, per)
    got = _forward_level("one pass", tgts[1], tgts[1].packed, toks, rows, mask_base, first, n, k, per)
    assert (got[0] >= 0).all()
    _same_level(tgts, want, got, shape, first, n)


@pytest.mark.parametrize("lanes", [2, 3, 4])
def test_a_wide_level_keeps_to_the_compute_units_of_its_lanes(lanes, monkeypatch):
    """The pass whose kernels spread over the whole GPU is taken only where the lanes (of 64 workgroups) have all of it."""
    from paper_2508_04462_amd import binding

    tgts, want, toks, rows, mask_base, _ = _level_twice(MID, 28, 70, 80, 100, 5, lanes)
    one_pass, calls = binding.card_draft_level_wide, []
    monkeypatch.setattr(binding, "card_draft_level_wide", lambda *a: calls.append(1) or one_pass(*a))
    res = tgts[1].draft_level_wide(70, toks, [71] * 100, 80, rows, mask_base, 5)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert len(calls) == (1 if lanes * 64 == cus else 0)
    _same_level(tgts, want, (res["topk_tokens"].cpu(), res["topk_probs"].cpu()), MID, 80, 100)


def test_lanes_are_refused_where_no_share_of_the_gpu_was_given():
    import paper_2508_04462_amd as card

    with pytest.raises(ValueError):  # (a small model's own choice of a grid is no such share)
        card.Target(TINY, 128).enable_lanes(2)


@pytest.mark.parametrize("n", [5, 12, 32, 100])
def test_draft_calls_give_no_candidates_for_weights_packed_for_another_grid(n):
    """As a verification step reports it: a level in one call (up to 32 rows), in pieces, in one pass."""
    import paper_2508_04462_amd as card
    from paper_2508_04462_amd.synthetic import load_synthetic_weights

    tgts, want, toks, rows, mask_base, _ = _level_twice(MID, 27, 70, 80, n, 5, 2)
    tgt, other = tgts[1], card.Target(MID, 320, grid_wgs=128)
    load_synthetic_weights(other, MID, 27, 0.2)
    for route in ("call", "pieces", "one pass")[n > 32:]:
        tk, tp = _forward_level(route, tgt, other.packed, toks, rows, mask_base, 80, n, 5)
        assert (tk == -1).all() and (tp == 0).all()
        tk, tp = _forward_level(route, tgt, tgt.packed, toks, rows, mask_base, 80, n, 5)
        assert (tk >= 0).all() and (tp > 0).all()
        if route == "pieces":
            assert torch.equal(tk, want[0]) and torch.equal(tp, want[1])


def test_a_wide_level_with_a_refused_piece_leaves_nothing_running():
    """The pieces in front of a refused one work on tensors of the call: it ends behind them."""
    import paper_2508_04462_amd as card

    tgts, _, toks, rows, mask_base, pieces = _level_twice(MID, 25, 70, 80, 100, 5, 2)
    assert len(pieces) == 4 and tgts[1]._level_ws is None  # (side by side: one pass is refused before anything runs)
    short = [row[:3] for row in rows]  # 96 slots from mask_base = 64: the last pieces' lie behind them
    with pytest.raises(card.CardError) as e:
        tgts[1].draft_level_wide(70, toks, [71] * 100, 80, short, mask_base, 5)
    assert e.value.status == card.CARD_ERANGE
    assert all(st.query() for st in tgts[1]._lane_streams)
    res = tgts[1].draft_level_wide(70, toks, [71] * 100, 80, rows, mask_base, 5)
    assert (res["topk_tokens"] >= 0).all()


@pytest.mark.parametrize("n", [8, 13, 29])
def test_a_chain_forwarded_as_tree_rows_equals_the_verify_step_bit_for_bit(n):
    """Tree rows whose mask is the plain causal chain (row i sees the context and rows 0..i, slots
    = positions) are the rows of a verification step: card_draft_level must then give the logits
    and keys of card_verify bit for bit - the tree mask, the separate positions and slots change
    what a row sees, never how its sums are taken."""
    import paper_2508_04462_amd as card
    from paper_2508_04462_amd.synthetic import load_synthetic_weights

    shape, seed, ctx_len = MID, 31, 75
    tgt = card.Target(shape, 192, max_r=32)
    load_synthetic_weights(tgt, shape, seed, 0.2)
    toks = ci.uniform_tokens(seed, "ctx_tokens", 0, ctx_len + n, shape.vocab).tolist()
    tgt.prefill(toks[:ctx_len])
    ref = tgt.verify(ctx_len, -1, toks[ctx_len:], want_logits=True)
    k_ref, v_ref = tgt.kv_gather(shape.n_layers - 1, ctx_len, n)
    mask_base = ctx_len // 16 * 16
    words = (ctx_len + n - mask_base + 31) // 32
    rows, prev = [], None
    for i in range(n):
        st, row = card.card_tree_mask_level(prev, [-1 if i == 0 else 0], ctx_len + i, ctx_len, mask_base, words)
        rows.append(row[0])
        prev = row
    res = tgt.draft_level(ctx_len, toks[ctx_len:], [ctx_len + i for i in range(n)], ctx_len, rows, mask_base, 4, want_logits=True)
    assert torch.equal(res["logits"], ref["logits"])
    k, v = tgt.kv_gather(shape.n_layers - 1, ctx_len, n)
    assert torch.equal(k, k_ref) and torch.equal(v, v_ref)
    # the fused top-k's first entry is the arg-max the verify step reports
    assert res["topk_tokens"][:, 0].tolist() == ref["row_argmax"]
