"""Batches of many requests (MI355X only).

Every scoring and selecting workgroup derives the scoring ranges from the
lengths of all requests: of up to 64 by one scan, of up to 512 by blocks of
consecutive requests, and above that from the stored positions instead.
Ragged lengths with empty requests at both ends and runs of them between, on
both sides of each edge, through every path that scores: score_keys against
the oracle, and the sets of the others, exactly the oracle's on those scores.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2607_26475_amd as ckv
from helpers import ATOL_OUT, SCALE, check_scores, device, oracle_attn_over, orc, u16

pytestmark = pytest.mark.gpu

D = 128
CASES = [  # requests, KV heads, group size, stored rows, k
    (64, 1, 4, 300, 40), (65, 2, 2, 300, 40), (130, 1, 1, 1100, 64), (512, 2, 4, 161, 32),
    (513, 1, 8, 300, 40), (700, 2, 4, 97, 32), (1100, 8, 2, 64, 16)]


def _lens(B, n):
    rng = np.random.default_rng(B)
    lens = rng.integers(0, n + 1, size=B)
    lens[[0, 1, B - 1, B // 2]] = 0
    lens[B // 3:B // 3 + min(B // 4, 70)] = 0
    lens[[2, B // 2 + 1, B - 2]] = n
    lens[[3, 4]] = 1, 32
    return lens.astype(np.int32)


class Inputs:
    def __init__(self, B, H, G, n, k):
        dev = device()
        g = torch.Generator(device=dev)
        g.manual_seed(B * 7 + n)
        rn = lambda *s: torch.randn(s, generator=g, device=dev, dtype=torch.bfloat16)  # noqa: E731
        self.B, self.H, self.G, self.n, self.k, self.dev = B, H, G, n, k, dev
        self.q, self.q2 = rn(B, H * G, D), rn(B, H * G, D)
        self.K, self.V = rn(B, H, n, D), rn(B, H, n, D)
        self.lens = _lens(B, n)
        self.dl = torch.from_numpy(self.lens).to(dev)
        self.shape = ckv.shape_for(B, H * G, H, n)
        self.rn = rn

    def sets(self):
        return (torch.full((self.B, self.H, self.k), -9, dtype=torch.int32, device=self.dev),
                torch.full((self.B, self.H), -9, dtype=torch.int32, device=self.dev))

    def out(self):
        return torch.full((self.B, self.H * self.G, D), float("nan"), device=self.dev)

    def ws(self, entry):
        w = ckv.workspace(self.shape, self.k, entry)
        w.fill_(0xA5)
        return w

    def scores(self, q):
        s = torch.full((self.B, self.H, self.n), float("nan"), device=self.dev)
        ckv.score_keys(self.shape, q, self.K, self.dl, SCALE, s)
        return s.cpu().numpy()

    def want(self, scores):
        o = orc()
        so = o.shape(self.B, self.H * self.G, self.H, D, self.n)
        return o.select_topk(so, scores.astype(np.float64), self.lens, self.k, nthreads=8)


def _equal(got, want):
    np.testing.assert_array_equal(got[1].cpu().numpy(), want[1])
    np.testing.assert_array_equal(got[0].cpu().numpy(), want[0])


@pytest.mark.parametrize("B,H,G,n,k", CASES)
def test_many_requests(B, H, G, n, k):
    print("many requests", B, H, G, n, k, flush=True)
    t = Inputs(B, H, G, n, k)
    o = orc()
    so = o.shape(B, H * G, H, D, n)
    Kh = u16(t.K)
    S, S2 = t.scores(t.q), t.scores(t.q2)
    check_scores(S, o.score_keys(so, u16(t.q), Kh, t.lens, SCALE, nthreads=8), u16(t.q), Kh,
                 t.lens, G)
    want, want2 = t.want(S), t.want(S2)
    ref = oracle_attn_over(so, u16(t.q), Kh, u16(t.V), *want, k)
    d_idx, d_n = torch.from_numpy(want[0]).to(t.dev), torch.from_numpy(want[1]).to(t.dev)

    same, out = t.sets(), t.out()
    ckv.critical_kv_attn(t.shape, t.q, None, t.K, t.dl, k, SCALE, t.K, t.V, ckv.SRC_DEVICE, None,
                         None, None, *same, out, t.ws(ckv.ENTRY_CRITICAL_KV_ATTN))
    _equal(same, want)
    assert np.abs(out.cpu().numpy() - ref).max() <= ATOL_OUT

    pipe, out = t.sets(), t.out()
    ckv.critical_kv_attn(t.shape, t.q, t.q2, t.K, t.dl, k, SCALE, t.K, t.V, ckv.SRC_DEVICE, None,
                         None, d_n, *pipe, out, t.ws(ckv.ENTRY_CRITICAL_KV_ATTN), idx_in=d_idx)
    _equal(pipe, want2)
    assert np.abs(out.cpu().numpy() - ref).max() <= ATOL_OUT

    for second in (t.q2, None):  # two queries, one
        kb, vb = torch.zeros((B, H, k, D), dtype=torch.bfloat16, device=t.dev), None
        vb = torch.zeros_like(kb)
        true, nxt, out = t.sets(), t.sets(), t.out()
        hits = torch.full((B, H), -9, dtype=torch.int32, device=t.dev)
        pred, n_pred = torch.full_like(d_idx, -1), torch.zeros_like(d_n)
        ckv.corrected_attn(t.shape, t.q, second, t.K, t.dl, k, SCALE, t.K, t.V, ckv.SRC_DEVICE,
                           pred, n_pred, kb, vb, *true, hits, *nxt, out,
                           t.ws(ckv.ENTRY_CORRECTED_ATTN))
        _equal(true, want)
        _equal(nxt, want2 if second is not None else want)
        assert int(hits.abs().max()) == 0
        assert np.abs(out.cpu().numpy() - ref).max() <= ATOL_OUT

    chunk = 4
    cmax, cl = -(-n // chunk), -(-t.lens // chunk)
    marks = t.rn(B, H, cmax, D)
    cs = ckv.shape_for(B, H * G, H, cmax)
    sc = torch.full((B, H, cmax), float("nan"), device=t.dev)
    ckv.score_keys(cs, t.q2, marks, torch.from_numpy(cl).to(t.dev), SCALE, sc)
    picked = o.select_topk(o.shape(B, H * G, H, D, cmax), sc.cpu().numpy().astype(np.float64), cl,
                           k // chunk, nthreads=8)
    rows = t.sets()
    c_idx = torch.full((B, H, k // chunk), -9, dtype=torch.int32, device=t.dev)
    c_n = torch.full((B, H), -9, dtype=torch.int32, device=t.dev)
    ckv.select_chunks(t.shape, chunk, t.q2, marks, t.dl, k, SCALE, c_idx, c_n, *rows,
                      t.ws(ckv.ENTRY_CRITICAL_KV_ATTN))
    _equal((c_idx, c_n), picked)


@pytest.mark.parametrize("two", [False, True], ids=["plain", "two_tokens"])
@pytest.mark.parametrize("B", [65, 513])
def test_many_requests_loop(B, two):
    """Three layers in place: a layer's selection runs in the next one's launch."""
    print("many requests, loop", B, two, flush=True)
    t = Inputs(B, 2, 4, 300, 32)
    S = t.scores(t.q2)
    want = t.want(S)
    prev = t.want(t.scores(t.q))
    d_prev = [torch.from_numpy(x).to(t.dev) for x in prev]
    layers = []
    for _ in range(3):
        idx, n_sel = t.sets()
        d = {"q_att": t.q, "q_sel": t.q2, "k_score": t.K, "k_src": t.K, "v_src": t.V,
             "idx_prev": d_prev[0], "n_sel_prev": d_prev[1], "idx_next": idx,
             "n_sel_next": n_sel, "out": t.out()}
        if two:
            d.update(k_local=t.rn(B, 2, 2, D), v_local=t.rn(B, 2, 2, D), out_spec=t.out())
        layers.append(d)
    p = ckv.Pipeline()
    p.step(t.shape, layers, t.dl, t.k, SCALE, ckv.SRC_DEVICE, None, None,
           t.ws(ckv.ENTRY_DECODE_STEP), None, 0)
    torch.cuda.synchronize()
    p.close()
    so = orc().shape(B, 8, 2, D, t.n)
    ref = oracle_attn_over(so, u16(t.q), u16(t.K), u16(t.V), *prev, t.k)
    for d in layers:
        _equal((d["idx_next"], d["n_sel_next"]), want)
        if not two:
            assert np.abs(d["out"].cpu().numpy() - ref).max() <= ATOL_OUT


@pytest.mark.parametrize("n", [65537, 65540])
def test_many_long_requests(n):
    """Stored positions under claims: the scoring of one-launch pipelined calls
    past 65536 positions, half as ranges and half as claims."""
    print("many long requests", n, flush=True)
    t = Inputs(513, 1, 4, n, 64)
    want = t.want(t.scores(t.q2))
    idx_in = torch.zeros((513, 1, 64), dtype=torch.int32, device=t.dev)
    n_in = torch.zeros((513, 1), dtype=torch.int32, device=t.dev)
    ws, got, out = t.ws(ckv.ENTRY_CRITICAL_KV_ATTN), t.sets(), t.out()
    for _ in range(2):
        ckv.critical_kv_attn(t.shape, t.q, t.q2, t.K, t.dl, t.k, SCALE, t.K, t.V, ckv.SRC_DEVICE,
                             None, None, n_in, *got, out, ws, idx_in=idx_in)
        _equal(got, want)
        got[0].fill_(-9)
    assert float(out.abs().max()) == 0.0  # nothing was selected one step earlier
