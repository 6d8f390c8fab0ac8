"""Decoder steps from a state that the caller wrote: the state buffer holds fp32 h, c and feed, which a program may
keep, edit and step from more than once, so a step leaves it as it is."""

import numpy as np
import pytest
import torch

import workloads as W
from oracle import onmt_oracle as O
from paper_1805_11462_amd import _lib
from paper_1805_11462_amd.translator import _ptr, _stream
from ._gpu import translator_for, with_workload

pytestmark = pytest.mark.gpu


class Step:
    """A one-batch model and the state after its first step, as the caller's own to edit."""

    def __init__(self, wdtype, hidden, layers, B, K, weights=None, **kw):
        self.w = with_workload(W.get("tiny"), hidden=hidden, emb=32, enc_layers=layers, dec_layers=layers,
                               wdtype=wdtype, **kw)
        self.weights = weights or W.make_weights(self.w)
        self.tr = translator_for(self.w, self.weights)
        self.B, self.K, self.S, self.N = B, K, 5, B * K
        rng = np.random.default_rng(7)
        self.rng = rng
        src = torch.from_numpy(rng.integers(4, self.w.src_vocab, (B, self.S)).astype(np.int32)).cuda()
        self.lens = torch.from_numpy(rng.integers(1, self.S + 1, B).astype(np.int32)).cuda()
        self.ws = self.tr.encode(src, self.lens)
        self.tok = torch.from_numpy(rng.integers(4, self.w.tgt_vocab, self.N).astype(np.int32)).cuda()
        self.par = torch.from_numpy((np.arange(self.N) // K * K + rng.integers(0, K, self.N)).astype(np.int32)).cuda()
        st = self.tr.decode_init(self.ws, B, self.S, K)
        self.state = self.tr.decode_step(self.ws, B, self.S, K, st, self.tok, None, mode=1)[0]
        self.h, self.c, self.feed = self.tr.state_views(self.state, self.N)

    def step(self):
        return self.tr.decode_step(self.ws, self.B, self.S, self.K, self.state, self.tok, self.par, mode=1)

    def noalloc(self):
        out, N, K = self.tr.new_state(self.N), self.N, self.K
        logp = torch.empty(N, K, dtype=torch.float32, device="cuda")
        ids = torch.empty(N, K, dtype=torch.int32, device="cuda")
        _lib.check(self.tr.lib.onmt_decode_step_noalloc(
            self.tr.handle, _ptr(self.ws), self.B, self.S, K, _ptr(self.state), _ptr(out), _ptr(self.tok),
            _ptr(self.par), 1, _ptr(logp), _ptr(ids), None, None, _stream()))
        return out, logp, ids


@pytest.mark.parametrize("wdtype,hidden,layers,B,K", [
    ("fp32", 64, 1, 3, 2), ("fp32", 100, 3, 17, 1), ("bf16", 100, 2, 7, 5), ("bf16", 104, 2, 7, 5),
])
def test_a_step_leaves_its_input_state_as_it_is(wdtype, hidden, layers, B, K):
    s = Step(wdtype, hidden, layers, B, K)
    print(f"[case] input state kept {wdtype} H{hidden} L{layers} {B}x{K}", flush=True)
    for x in (s.h, s.c, s.feed):
        x.copy_(torch.from_numpy(s.rng.uniform(-1, 1, tuple(x.shape)).astype(np.float32)))
    before = s.state.clone()
    a = s.step()
    assert torch.equal(s.state, before)
    n = s.noalloc()
    assert torch.equal(s.state, before)
    b = s.step()                         # and the same state gives the same step again
    for other in (b, n):
        for x, y in zip(s.tr.state_views(a[0], s.N), s.tr.state_views(other[0], s.N)):
            assert torch.equal(x, y)
        assert torch.equal(a[1], other[1]) and torch.equal(a[2], other[2])
    s.tr.close()


def _exact(s):
    """The step in 64 bits with torch: (h, c, feed)."""
    t = {k: torch.from_numpy(v).cuda().double() for k, v in s.weights.items()}
    par, H = s.par.long(), s.w.hidden
    h, c, feed = (x.double()[..., par, :] for x in (s.h, s.c, s.feed))
    x = torch.cat([t["E_tgt"][s.tok.long()], feed], 1)
    hs, cs = [], []
    for l in range(s.w.dec_layers):
        z = torch.cat([x, h[l]], 1) @ t[f"dec{l}_W"].t().contiguous() + t[f"dec{l}_b"]
        i, f, g, o = z.chunk(4, 1)
        cs.append(torch.sigmoid(f) * c[l] + torch.sigmoid(i) * torch.tanh(g))
        x = torch.sigmoid(o) * torch.tanh(cs[-1])
        hs.append(x)
    mem, keys, _, _ = (v.double() for v in s.tr.enc_views(s.ws, s.B, s.S))
    e = torch.bmm(x.reshape(s.B, s.K, H), keys.transpose(1, 2).contiguous())
    off = torch.arange(s.S, device="cuda")[None, None, :] >= s.lens[:, None, None]
    ctx = torch.bmm(torch.softmax(e.masked_fill(off, -float("inf")), -1), mem).reshape(s.N, H)
    return torch.stack(hs), torch.stack(cs), torch.tanh(torch.cat([ctx, x], 1) @ t["W_c"].t().contiguous())


@pytest.mark.parametrize("wdtype,layers,log2", [
    ("fp32", 1, -100), ("fp32", 1, -30), ("fp32", 1, 16), ("fp32", 1, 100), ("fp32", 2, 23), ("fp32", 3, -23),
    ("fp32", 3, 16), ("bf16", 2, 16), ("bf16", 2, -23),
])
def test_states_of_any_size(wdtype, layers, log2):
    # h and feed of size 2^log2 (every third row 2^9 smaller) against weights that bring their products back to size 1,
    # so that an error of the operands reaches the outputs
    hidden, emb = 100, 32
    base = Step(wdtype, hidden, layers, 7, 5)
    weights = dict(base.weights)
    base.tr.close()
    for l in range(layers):
        W_l = weights[f"dec{l}_W"].copy()
        W_l[:, emb if l == 0 else hidden:] *= np.float32(2.0) ** -log2
        weights[f"dec{l}_W"] = W_l
    s = Step(wdtype, hidden, layers, 7, 5, weights=weights)
    print(f"[case] states of size 2^{log2} {wdtype} L{layers}", flush=True)
    size = np.float32(2.0) ** np.where(np.arange(s.N) % 3 == 0, log2 - 9, log2).astype(np.float32)
    for x in (s.h, s.feed):
        v = s.rng.uniform(-1, 1, tuple(x.shape)).astype(np.float32) * size[:, None]
        x.copy_(torch.from_numpy(v))
    s.c.copy_(torch.from_numpy(s.rng.uniform(-1, 1, tuple(s.c.shape)).astype(np.float32)))
    got = s.tr.state_views(s.step()[0], s.N)
    # sums of 200 products of size <= 0.1 with operands good to 2^-22 each, then functions of slope <= 1 (twice over
    # the layers and the output)
    for x, y in zip(got, _exact(s)):
        assert (x.double() - y).abs().max().item() <= 2e-6 * (1 + layers)
    s.tr.close()


@pytest.mark.parametrize("spike", [5e3, 1e6, 3e38])
def test_single_large_elements_saturate_their_gates(spike):
    # one element of a row far beyond the rest: the gates it reaches saturate by its sign, the row stays finite
    s = Step("fp32", 100, 2, 7, 5)
    print(f"[case] spike {spike}", flush=True)
    for l in range(2):
        s.h[l, torch.arange(s.N), torch.arange(s.N) % 100] = spike
    s.feed[3, 7] = -spike
    got = s.tr.state_views(s.step()[0], s.N)
    # |w| >= 1e-5 on a spike of 5e3 leaves no gate between the states beyond the rounding of its product (2^-21 of it)
    near = 2.0 ** -21 * 0.1 * spike
    for x, y in zip(got, _exact(s)):
        assert torch.isfinite(x).all()
        d = (x.double() - y).abs()
        assert d.max().item() <= (near if near < 1 else 2) and (d > 1e-4).double().mean().item() <= 1e-3
    s.tr.close()


@pytest.mark.parametrize("what", ["state", "weight", "embedding"])
@pytest.mark.parametrize("wdtype,layers", [("fp32", 1), ("fp32", 3), ("bf16", 2)])
def test_an_infinite_element_saturates_its_gates(what, wdtype, layers):
    base = Step(wdtype, 100, layers, 7, 5)
    weights = {k: v.copy() for k, v in base.weights.items()}
    base.tr.close()
    if what == "weight":          # units 3 and 8 of every layer: input gate by the first column of [below], forget by h
        for l in range(layers):
            weights[f"dec{l}_W"][3, 32 if l == 0 else 0] = np.inf
            weights[f"dec{l}_W"][108, -5] = -np.inf
    s = Step(wdtype, 100, layers, 7, 5, weights=weights)
    print(f"[case] infinite {what} {wdtype} L{layers}", flush=True)
    if what == "state":
        rows = torch.arange(s.N)
        s.feed[rows[::2], 7] = float("inf")                   # one infinity per row of a layer's product
        s.h[0, rows[1::2], 99] = -float("inf")
        s.h[1:, rows, rows % 100] = float("inf")
    if what == "embedding":
        s.weights = dict(weights)
        s.weights["E_tgt"][s.tok[0].item(), 9] = np.inf       # (also of the first step's token: that state is kept)
        state = s.state.clone()
        s.tr.close()
        s.tr = translator_for(s.w, s.weights)
        s.ws = s.tr.encode(torch.full((s.B, s.S), 5, dtype=torch.int32, device="cuda"), s.lens)
        s.state = state
        s.h, s.c, s.feed = s.tr.state_views(state, s.N)
    for x, y in zip(s.tr.state_views(s.step()[0], s.N), _exact(s)):
        assert torch.isfinite(y).all()
        assert (x.double() - y).abs().max().item() <= 1e-5 * (1 + layers)
    s.tr.close()


@pytest.mark.parametrize("wdtype", ["fp32", "bf16"])
def test_an_infinite_source_embedding_saturates_its_gates(wdtype):
    # a 2-layer encoder over 136-wide embeddings (five K blocks, no multiple of the projection's stages)
    w = with_workload(W.get("tiny"), emb=136, hidden=64, enc_layers=2, dec_layers=2, wdtype=wdtype)
    weights = W.make_weights(w)
    weights["E_src"][[6, 9], [135, 3]] = np.inf, -np.inf
    tr = translator_for(w, weights)
    print(f"[case] infinite embedding {wdtype}", flush=True)
    src = np.random.default_rng(3).integers(4, 12, (5, 7)).astype(np.int32)
    lens = np.array([7, 6, 7, 1, 3], np.int32)
    ws = tr.encode(torch.from_numpy(src).cuda(), torch.from_numpy(lens).cuda())
    mem = tr.enc_views(ws, 5, 7)[0].cpu().numpy()
    src[np.arange(7)[None, :] >= lens[:, None]] = W.PAD_ID
    with np.errstate(over="ignore", invalid="ignore"):
        want = O.encode(O.model_from(w, weights), src, lens).memory
    assert np.isfinite(want).all()
    np.testing.assert_allclose(mem, want, atol=1e-5, rtol=0)
    tr.close()


@pytest.mark.parametrize("wdtype,hidden", [("fp32", 100), ("bf16", 104)])
def test_steps_of_edited_states_can_be_captured(wdtype, hidden):
    # steps captured once and replayed on states that change between the replays: copies and powers of two are made
    # in the graph, not kept from the capture
    s = Step(wdtype, hidden, 2, 7, 5)
    print(f"[case] captured steps {wdtype} H{hidden}", flush=True)
    tr = s.tr
    _lib.check(tr.lib.onmt_set_validation(tr.handle, _lib.ONMT_VALIDATE_DEVICE))
    first = s.state.clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        s.step(), s.noalloc()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        a, n = s.step(), s.noalloc()
    for size in (1.0, 1e6, 1e-9, 1.0):
        s.state.copy_(first)
        if wdtype == "fp32":
            s.h *= size
            s.feed *= size
        graph.replay()
        torch.cuda.synchronize()
        want = s.step()
        for got in (a, n):
            for x, y in zip(tr.state_views(got[0], s.N), tr.state_views(want[0], s.N)):
                assert torch.equal(x, y)
            assert torch.equal(got[1], want[1]) and torch.equal(got[2], want[2])
    tr.close()
