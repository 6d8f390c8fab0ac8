"""Decoder steps from a state that the caller wrote: the state buffer holds fp32 h, c and feed, which a program may
keep, edit and step from more than once, so a step leaves it as it is."""

import numpy as np
import pytest
import torch

import workloads as W
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
