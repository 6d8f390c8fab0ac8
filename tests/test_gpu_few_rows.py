"""The few-row products (decoder layers, attentional output) at the sizes where their tiles change: rows around the
16-row blocks and each tile height, hidden sizes that end inside an 8-unit group or a 32-column block, one to three
layers, rows gathered through a parent map, and a caller's own fp32 state."""

import numpy as np
import pytest
import torch

import workloads as W
from oracle import onmt_oracle as O
from ._gpu import translator_for, with_workload

pytestmark = pytest.mark.gpu


def _exact_step(w, weights, mem, keys, lens, h, c, feed, tok, par, K):
    """One decoder step in 64 bits with torch: (h, c, feed)."""
    t = {k: torch.from_numpy(v).cuda().double() for k, v in weights.items()}
    x = torch.cat([t["E_tgt"][tok], feed[par]], 1)
    hs, cs = [], []
    for l in range(w.dec_layers):
        z = torch.cat([x, h[l][par]], 1) @ t[f"dec{l}_W"].t().contiguous() + t[f"dec{l}_b"]
        i, f, g, o = z.chunk(4, 1)
        cl = torch.sigmoid(f) * c[l][par] + torch.sigmoid(i) * torch.tanh(g)
        x = torch.sigmoid(o) * torch.tanh(cl)
        hs.append(x)
        cs.append(cl)
    B, S, H = mem.shape
    e = torch.bmm(x.reshape(B, K, H), keys.transpose(1, 2).contiguous())
    off = torch.arange(S, device="cuda")[None, None, :] >= lens[:, None, None]
    a = torch.softmax(e.masked_fill(off, -float("inf")), -1)
    ctx = torch.bmm(a, mem).reshape(B * K, H)
    return torch.stack(hs), torch.stack(cs), torch.tanh(torch.cat([ctx, x], 1) @ t["W_c"].t().contiguous())


@pytest.mark.parametrize("wdtype,hidden,layers,B,K", [
    ("fp32", 36, 1, 1, 1), ("fp32", 64, 2, 5, 3), ("fp32", 100, 1, 4, 4), ("fp32", 100, 3, 17, 1),
    ("fp32", 516, 1, 13, 5), ("fp32", 500, 2, 27, 3), ("fp32", 500, 1, 16, 10), ("fp32", 500, 2, 23, 7),
    ("fp32", 500, 1, 32, 10), ("fp32", 68, 1, 81, 4), ("fp32", 1000, 1, 33, 5),
    ("bf16", 36, 1, 1, 1), ("bf16", 100, 2, 7, 5), ("bf16", 500, 2, 64, 1), ("bf16", 1000, 2, 64, 5),
    ("bf16", 1024, 1, 513, 1), ("bf16", 1000, 1, 32, 4), ("bf16", 104, 1, 81, 5),
    ("bf16", 1000, 2, 128, 4), ("bf16", 500, 1, 205, 5),
    *(("fp32", 68, 1, 3, k) for k in (6, 8, 9, 11, 12, 13, 14, 15, 16)),     # one instantiation per beam width
])
@pytest.mark.parametrize("own_state", [False, True, 1000])     # 1000: h and feed of up to 3000
def test_decoder_layers(wdtype, hidden, layers, B, K, own_state):
    if own_state and wdtype == "bf16" and hidden % 8 == 0:
        pytest.skip("such models read the operand copies their producer left beside h and feed")
    w = with_workload(W.get("tiny"), hidden=hidden, emb=32, enc_layers=layers, dec_layers=layers, wdtype=wdtype)
    weights = W.make_weights(w)
    tr = translator_for(w, weights)
    print(f"[case] few rows {wdtype} H{hidden} L{layers} B{B} K{K} own_state={own_state}", flush=True)
    rng = np.random.default_rng(7)
    S, N = 5, B * K
    src = torch.from_numpy(rng.integers(4, w.src_vocab, (B, S)).astype(np.int32)).cuda()
    lens = torch.from_numpy(rng.integers(1, S + 1, B).astype(np.int32)).cuda()
    ws = tr.encode(src, lens)
    st = tr.decode_init(ws, B, S, K)
    tok = torch.from_numpy(rng.integers(4, w.tgt_vocab, N).astype(np.int32)).cuda()
    par = torch.from_numpy((np.arange(N) // K * K + rng.integers(0, K, N)).astype(np.int32)).cuda()
    st = tr.decode_step(ws, B, S, K, st, tok, None, mode=1)[0]
    h, c, feed = tr.state_views(st, N)
    if own_state:
        for x in (h, c, feed):
            big = 1 if x is c else int(own_state)
            x.copy_(torch.from_numpy(big * rng.uniform(-3, 3, tuple(x.shape)).astype(np.float32)))
    h, c, feed = h.double(), c.double(), feed.double()
    got = tr.decode_step(ws, B, S, K, st, tok, par, mode=1)[0]
    mem, keys, _, _ = tr.enc_views(ws, B, S)
    want = _exact_step(w, weights, mem.double(), keys.double(), lens.long(), h, c, feed, tok.long(), par.long(), K)
    for x, y in zip(tr.state_views(got, N), want):
        # pre-activations sum 2 hidden + 32 products of size <= 0.3 to 2^-22 each, then pass through functions of
        # slope <= 1 (twice over the layers and the output); a c of size 4 keeps 2^-22 of itself; with the size of the
        # inputs the error of their sums grows
        assert (x.double() - y).abs().max().item() <= 2e-6 * (1 + layers) * 3 ** bool(own_state) * max(1, int(own_state))
    tr.close()


def test_zero_states_stay_zero():
    w = with_workload(W.get("tiny"), batch=3)
    weights = {k: np.zeros_like(v) for k, v in W.make_weights(w).items()}
    tr = translator_for(w, weights)
    src, lens = W.make_batch(w, batch=3)
    buf = tr.search_buffers(3, src.shape[1], 2, 4)
    tr.beam_search(torch.from_numpy(src).cuda(), torch.from_numpy(lens).cuda(), buf)
    m = O.model_from(w, weights)
    for b in range(3):
        n = int(buf["len"][b])
        toks = [int(x) for x in buf["tok"][b, :n].cpu()]
        ref = O.score_forced(m, src[b], lens[b], toks)
        np.testing.assert_allclose(buf["tok_logp"][b, :n].cpu().numpy(), ref, atol=2e-6)
    tr.close()


@pytest.mark.parametrize("log2", [-6, -14, -24])
def test_tiny_states_keep_the_precision_of_their_format(log2):
    # the weights that make the memory and h are small, those that multiply them large, so that an error of the operands
    # reaches the keys and the feed: operands are good to 2^-22 of the value or an absolute 2^-40 (a product doubles
    # what it keeps of the first, for the weights' own terms)
    w = with_workload(W.get("tiny"), batch=5)
    weights = {k: v.copy() for k, v in W.make_weights(w).items()}
    H, scale = w.hidden, np.float32(2.0) ** log2
    for k in ("enc0_fwd_W", "enc0_fwd_b", "dec0_W", "dec0_b"):
        weights[k] *= scale
    weights["W_a"] = weights["W_a"] / scale
    weights["W_c"][:, H:] /= scale                       # columns [context | h]
    tr = translator_for(w, weights)
    print(f"[case] tiny states 2^{log2}", flush=True)
    rng = np.random.default_rng(7)
    B, S, K = 5, 6, 2
    src = torch.from_numpy(rng.integers(4, w.src_vocab, (B, S)).astype(np.int32)).cuda()
    lens = torch.full((B,), S, dtype=torch.int32, device="cuda")
    ws = tr.encode(src, lens)
    mem, keys, _, _ = (x.double() for x in tr.enc_views(ws, B, S))
    assert 0 < mem.abs().max() < 4 * scale               # the encoder's outputs did shrink
    t = {k: torch.from_numpy(v).cuda().double() for k, v in weights.items()}

    def operand(x):
        return 2.0 ** -21 * x.abs() + 2.0 ** -40

    def close(got, x, W_, err):
        want, size = x @ W_.t().contiguous(), W_.abs().t().contiguous()
        sums = 2.0 ** -22 * (x.abs() @ size)             # the accumulators' roundings, two per 32 products
        return (got - want).abs(), err @ size + sums + 2.0 ** -23 * want.abs()

    d, bound = close(keys, mem, t["W_a"], operand(mem))
    assert (d <= bound).all() and keys.abs().max() > 1e-3
    # the memory itself: sums of 96 products good to 2^-21 each, and functions that keep relative precision near 0
    enc = O.encode(O.model_from(w, weights), src.cpu().numpy(), lens.cpu().numpy())
    np.testing.assert_allclose(mem.cpu().numpy(), enc.memory, atol=2e-6 * float(mem.abs().max()), rtol=0)

    N = B * K
    tok = torch.from_numpy(rng.integers(4, w.tgt_vocab, N).astype(np.int32)).cuda()
    st, _, _, _, attn = tr.decode_step(ws, B, S, K, tr.decode_init(ws, B, S, K), tok, None, mode=1, want_attn=True)
    h, _, feed = (x.double() for x in tr.state_views(st, N))
    ctx = torch.bmm(attn.double().reshape(B, K, S), mem).reshape(N, H)
    x = torch.cat([ctx, h[0]], 1)
    err = operand(x) + 2.0 ** -22 * torch.cat([ctx.abs(), torch.zeros_like(h[0])], 1)    # (the context's own sum)
    size = t["W_c"].abs().t().contiguous()
    z = x @ t["W_c"].t().contiguous()
    bound = err @ size + 2.0 ** -22 * (x.abs() @ size) + 2e-7                            # slope <= 1; tanhf's own error
    assert ((feed - torch.tanh(z)).abs() <= bound).all() and feed.abs().max() > 1e-3
    tr.close()
