"""The vocabulary projection at the sizes where its tiles change: rows around the 16-row blocks and the row
tiles of each kernel, vocabularies that end inside a 128-column tile, hidden sizes that end inside a 32-wide K
block, beams of 1 (per-tile best candidate) and more (logits)."""

import numpy as np
import pytest
import torch

import workloads as W
from ._gpu import translator_for, with_workload

pytestmark = pytest.mark.gpu


def _step(tr, w, B, K, S=4, seed=3):
    rng = np.random.default_rng(seed)
    src = torch.from_numpy(rng.integers(4, w.src_vocab, (B, S)).astype(np.int32)).cuda()
    lens = torch.full((B,), S, dtype=torch.int32, device="cuda")
    tok = torch.from_numpy(rng.integers(4, w.tgt_vocab, B * K).astype(np.int32)).cuda()
    ws = tr.encode(src, lens)
    st = tr.decode_init(ws, B, S, K)
    full = tr.decode_step(ws, B, S, K, st, tok, None, mode=0)
    topk = tr.decode_step(ws, B, S, K, st, tok, None, mode=1)
    return full, topk


@pytest.mark.parametrize("wdtype,hidden,vocab,B,K", [
    ("fp32", 64, 517, 1, 1), ("fp32", 64, 1000, 1, 16), ("fp32", 100, 2049, 3, 11), ("fp32", 516, 517, 32, 1),
    ("fp32", 68, 1153, 13, 5), ("fp32", 500, 3000, 16, 4), ("fp32", 500, 3000, 5, 16), ("fp32", 64, 1280, 27, 3),
    ("fp32", 100, 1025, 161, 1), ("fp32", 132, 4100, 160, 2), ("fp32", 64, 517, 321, 1), ("fp32", 36, 2000, 209, 4),
    ("bf16", 64, 517, 1, 5), ("bf16", 104, 2049, 13, 5), ("bf16", 100, 1025, 49, 3), ("bf16", 516, 1153, 161, 1),
    ("bf16", 1024, 2000, 64, 5),
])
def test_generator_tiles(wdtype, hidden, vocab, B, K):
    emb = 32
    w = with_workload(W.get("tiny"), hidden=hidden, emb=emb, tgt_vocab=vocab, wdtype=wdtype, batch=B, beam=K)
    weights = W.make_weights(w, peaked=True)
    tr = translator_for(w, weights)
    print(f"[case] generator {wdtype} H{hidden} V{vocab} rows {B * K} K{K}", flush=True)
    (st, logp, _, lse, _), (_, tv, ti, lse1, _) = _step(tr, w, B, K)
    feed = tr.state_views(st, B * K)[2].double()
    Ws = torch.from_numpy(weights["W_s"]).cuda().double()
    bs = torch.from_numpy(weights["b_s"]).cuda().double()
    z = feed @ Ws.t().contiguous() + bs
    # operands carry 22 significant bits each, accumulators are rounded once per 32 products and term product;
    # the logsumexp's exponentials and logarithm are good to a few units of 1e-7
    size = feed.abs() @ Ws.abs().t().contiguous()
    bound = size * (2.0 ** -21 + (hidden / 32 + 4) * 2.0 ** -23) + (z.abs() + bs.abs()) * 2.0 ** -22 + 2e-6
    assert (((logp + lse[:, None]).double() - z).abs() <= bound + lse[:, None].abs().double() * 2.0 ** -22).all()
    assert ((lse.double() - torch.logsumexp(z, 1)).abs() <= bound.max(dim=1)[0]).all()
    # the top-K of the same logits, exactly: larger first, smaller id on ties
    assert torch.equal(lse, lse1)
    lp = logp.cpu().numpy()
    ids = np.argsort(-lp, axis=1, kind="stable")[:, :K]
    np.testing.assert_array_equal(ti.cpu().numpy(), ids)
    np.testing.assert_array_equal(tv.cpu().numpy(), np.take_along_axis(lp, ids, 1))
    tr.close()


def test_generator_rows_of_large_and_tiny_weights():
    # every row of the projection has its own power-of-two scale: rows 1e6 apart in size, a zero row and a row
    # with one large entry keep the precision of fp32
    w = with_workload(W.get("tiny"), tgt_vocab=300, batch=4, beam=2)
    weights = W.make_weights(w)
    scale = np.float32(10.0) ** np.linspace(-30, 6, 300).astype(np.float32)
    weights["W_s"] = (weights["W_s"] * scale[:, None]).astype(np.float32)
    weights["W_s"][7] = 0.0
    weights["W_s"][11, 5] = 3e4
    tr = translator_for(w, weights)
    print("[case] generator row scales", flush=True)
    (st, logp, _, lse, _), _ = _step(tr, w, 4, 2)
    feed = tr.state_views(st, 8)[2].double()
    Ws = torch.from_numpy(weights["W_s"]).cuda().double()
    z = feed @ Ws.t().contiguous() + torch.from_numpy(weights["b_s"]).cuda().double()
    size = feed.abs() @ Ws.abs().t().contiguous() + z.abs() + lse.double()[:, None].abs()
    assert (((logp + lse[:, None]).double() - z).abs() <= size * 2.0 ** -20 + 1e-6).all()
    tr.close()


@pytest.mark.parametrize("vocab,K", [
    (5, 5), (12, 12), (63, 16), (65, 5), (128, 2), (129, 3), (300, 12), (1000, 12), (1920, 16), (1921, 16),
])
@pytest.mark.parametrize("kind", ["peaked", "ties", "few"])
def test_top_k_with_fewer_tiles_than_k(vocab, K, kind):
    # vocabularies of at most 128 (K - 1) words (and one beyond): "ties" has logits of a few distinct values, "few" fewer
    # finite logits than K
    w = with_workload(W.get("tiny"), hidden=64, emb=32, tgt_vocab=vocab, batch=3, beam=K)
    weights = W.make_weights(w, peaked=True)
    if kind != "peaked":
        weights["W_s"] = np.zeros_like(weights["W_s"])
        weights["b_s"] = (np.arange(vocab) * 7 % 5).astype(np.float32)
    if kind == "few":
        weights["b_s"][np.arange(vocab) % max(2, vocab // 2) != 1] = -np.inf
    tr = translator_for(w, weights)
    print(f"[case] top-K of {vocab} words, K{K}, {kind}", flush=True)
    (_, logp, _, _, _), (_, tv, ti, _, _) = _step(tr, w, 3, K)
    lp = logp.cpu().numpy()
    ids = np.argsort(-lp, axis=1, kind="stable")[:, :K]
    want = np.take_along_axis(lp, ids, 1)
    ids = np.where(np.isfinite(want), ids, 0x7fffffff)       # no candidate
    np.testing.assert_array_equal(ti.cpu().numpy(), ids)
    np.testing.assert_array_equal(tv.cpu().numpy(), want)
    tr.close()


def test_batches_of_very_many_rows_keep_top_k_lists():
    # 32800 rows of 131072 logits would pass 16 GiB: the workspace holds per-tile top-K lists instead, filters included
    B, S, K, V = 2050, 4, 16, 131072
    w = with_workload(W.get("tiny"), hidden=36, emb=32, tgt_vocab=V, beam=K)
    tr = translator_for(w, W.make_weights(w, peaked=True))
    print(f"[case] lists for {B * K} rows of {V}", flush=True)
    assert 0 < tr.lib.onmt_step_ws_bytes(tr.handle, B, S, K) < 5 << 30
    (_, logp, _, lse, _), (_, tv, ti, lse1, _) = _step(tr, w, B, K)
    assert torch.equal(lse, lse1)
    for r0 in range(0, B * K, 4096):
        lp, v, i = logp[r0:r0 + 4096], tv[r0:r0 + 4096], ti[r0:r0 + 4096].long()
        assert torch.equal(torch.topk(lp, K, dim=1)[0], v) and torch.equal(torch.gather(lp, 1, i), v)
        i = i.sort(dim=1)[0]
        assert (i[:, 1:] > i[:, :-1]).all()
    del logp
    # the same sentences alone, whose logits fit: the same tokens under filters (margins of a peaked model are far
    # above rounding), their scores to a few roundings
    rng = np.random.default_rng(5)
    src = torch.from_numpy(rng.integers(4, w.src_vocab, (B, S)).astype(np.int32)).cuda()
    lens = torch.full((B,), S, dtype=torch.int32, device="cuda")
    free = tr.beam_search(src, lens, tr.search_buffers(B, S, K, 2))["tok"][:, 0]
    banned = tuple(int(x) for x in torch.unique(free)[:40].cpu() if x != W.EOS_ID)
    outs = []
    for s, n in ((src, lens), (src[-8:].contiguous(), lens[-8:].contiguous())):
        buf = tr.search_buffers(s.shape[0], S, K, 3, banned=banned, max_unk=0)
        tr.beam_search(s, n, buf)
        outs.append((buf["tok"][-8:].clone(), buf["raw"][-8:].clone()))
        assert not set(buf["tok"].flatten().tolist()) & (set(banned) | {W.UNK_ID})
    assert torch.equal(outs[0][0], outs[1][0])
    assert (outs[0][1] - outs[1][1]).abs().max() <= 2e-5
    tr.close()
