"""The encoder at the sizes where its routes and tiles change: sentences per step around the 16-row blocks and the
wavefront's limit (256), one to three layers and both directions, embedding, hidden and direction sizes that end
inside a 32-column block, batches whose longest sentence is shorter than S_max, embeddings far from 1 in size."""

import numpy as np
import pytest
import torch

import workloads as W
from oracle import onmt_oracle as O
from ._gpu import translator_for, with_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("wdtype,layers,bi,emb,hidden,B,S,attn,scale", [
    ("fp32", 1, False, 36, 68, 1, 1, "general", 1.0), ("fp32", 2, False, 36, 100, 3, 7, "general", 1.0),
    ("fp32", 3, False, 500, 64, 17, 5, "concat", 1.0), ("fp32", 2, False, 32, 36, 255, 4, "dot", 1.0),
    ("fp32", 2, False, 64, 100, 256, 3, "general", 1.0), ("fp32", 3, False, 36, 68, 257, 4, "general", 1.0),
    ("fp32", 2, True, 36, 72, 5, 6, "general", 1.0), ("fp32", 3, True, 100, 120, 33, 4, "concat", 1.0),
    ("fp32", 1, True, 4, 8, 2, 9, "dot", 1.0), ("fp32", 2, False, 36, 68, 9, 6, "general", 1e4),
    ("fp32", 2, True, 36, 72, 9, 6, "general", 1e-6), ("fp32", 1, False, 512, 500, 64, 10, "general", 1.0),
    ("bf16", 2, False, 40, 100, 3, 7, "general", 1.0), ("bf16", 3, True, 104, 120, 65, 4, "concat", 1.0),
    ("bf16", 2, False, 512, 1024, 256, 3, "general", 1.0), ("bf16", 2, True, 40, 72, 300, 3, "dot", 1.0),
    ("bf16", 1, False, 40, 36, 1, 30, "general", 1e3),
    ("bf16", 2, False, 40, 1000, 510, 3, "dot", 1.0),
])
@pytest.mark.parametrize("short", [False, True])
def test_encoder_rows(wdtype, layers, bi, emb, hidden, B, S, attn, scale, short):
    w = with_workload(W.get("tiny"), enc_layers=layers, dec_layers=layers, bidirectional=bi, emb=emb, hidden=hidden,
                      wdtype=wdtype, attn=attn)
    weights = W.make_weights(w)
    weights["E_src"] = W.round_bf16(weights["E_src"] * np.float32(scale)) if wdtype == "bf16" else \
        (weights["E_src"] * np.float32(scale)).astype(np.float32)
    tr = translator_for(w, weights)
    print(f"[case] encoder {wdtype} L{layers} bi{bi} E{emb} H{hidden} B{B} S{S} {attn} x{scale} short{short}", flush=True)
    rng = np.random.default_rng(11)
    top = max(1, S - 2) if short else S
    lens = rng.integers(1, top + 1, B).astype(np.int32)
    lens[0] = top
    src = rng.integers(4, w.src_vocab, (B, S)).astype(np.int32)      # ids past the lengths are ignored
    ws = tr.encode(torch.from_numpy(src).cuda(), torch.from_numpy(lens).cuda())
    mem, keys, fh, fc = (x.double().cpu().numpy() for x in tr.enc_views(ws, B, S))
    m = O.model_from(w, weights)
    clean = np.where(np.arange(S)[None, :] < lens[:, None], src, W.PAD_ID)
    enc = O.encode(m, clean, lens)
    # pre-activations carry 2^-21 of the sum of their products' sizes (embeddings of size 0.1 scale), the functions
    # behind them have slopes of at most 1; errors add up over the steps and layers
    tol = (2e-6 + 2.0 ** -21 * min(0.1 * scale, 10.0) * 0.1 * emb ** 0.5 * 4) * layers
    real = np.arange(S)[None, :] < lens[:, None]
    np.testing.assert_allclose(mem, enc.memory, atol=tol, rtol=0)
    assert (mem[~real] == 0).all()
    for l in range(layers):
        np.testing.assert_allclose(fh[l], enc.final_h[l], atol=tol, rtol=0)
        np.testing.assert_allclose(fc[l], enc.final_c[l], atol=tol * 4, rtol=1e-6)
    if attn != "dot":
        Wa = weights["W_a"].astype(np.float64)
        want = enc.memory @ (Wa if attn == "general" else Wa[:, hidden:]).T
        np.testing.assert_allclose(keys, want, atol=tol * 4 + 1e-6, rtol=0)
        assert (keys[~real] == 0).all()
    tr.close()


@pytest.mark.parametrize("wdtype,B,S", [
    ("fp32", 300, 250),       # two slices of the embedding operand, the second ragged
    ("bf16", 601, 250),       # half the bytes per row
    ("fp32", 4100, 256),      # all positions' embeddings would pass 4 GiB, the memory (0.5 GiB) does not
])
def test_wide_embeddings_are_projected_slice_by_slice(wdtype, B, S):
    w = with_workload(W.get("tiny"), emb=1024, hidden=64, wdtype=wdtype)
    tr = translator_for(w, W.make_weights(w))
    print(f"[case] embedding slices {wdtype} {B}x{S}", flush=True)
    rng = np.random.default_rng(5)
    lens = rng.integers(1, S + 1, B).astype(np.int32)
    pick = [0, 1, B // 2, B - 2, B - 1]
    lens[[0, B - 1]] = S
    src = rng.integers(4, w.src_vocab, (B, S)).astype(np.int32)

    def views(src, lens):
        ws = tr.encode(torch.from_numpy(src).cuda(), torch.from_numpy(lens).cuda())
        return [x.clone() for x in tr.enc_views(ws, *src.shape)]

    mem, keys, fh, fc = views(src, lens)
    # the same sentences alone: the same sums in other tiles, each good to 1e-6 (see above), so 2e-6 apart at most
    mem1, keys1, fh1, fc1 = views(np.ascontiguousarray(src[pick]), np.ascontiguousarray(lens[pick]))
    tol = 4e-6
    assert (mem[pick] - mem1).abs().max() <= tol and (keys[pick] - keys1).abs().max() <= tol
    assert (fh[:, pick] - fh1).abs().max() <= tol and (fc[:, pick] - fc1).abs().max() <= 4 * tol
    tr.close()
