"""Two queries scored in one pass over the keys (MI355X only).

The corrected entry selects the current token's set and the next step's from
one pass.  Every group size has its own placement of the two queries' head
rows in the matrix products; histograms go to slots (many units) or are added
(few units, long contexts); heavy ties exceed a selection's candidate list.
The caller may pass one query for both (the set is then written twice) and
may let the next step's sets take the place of the prediction, or of the
call's own sets and counts.  Sets against the oracle, outputs against the
oracle's attention over the sets.
"""
from __future__ import annotations

import dataclasses

import numpy as np
import pytest
import torch

import paper_2607_26475_amd as ckv
import synth
from helpers import (ATOL_OUT, SCALE, check_index_sets, device, make_prediction,
                     oracle_attn_over, orc, u16)

pytestmark = pytest.mark.gpu

CASES = [  # name, B, Hkv, G, stored rows, k, queries, next set in the prediction's place
    ("g1", 2, 2, 1, 1031, 96, 2, False),
    ("g2", 2, 2, 2, 1030, 96, 2, False),
    ("g4", 2, 2, 4, 4500, 256, 2, True),
    ("g8", 2, 2, 8, 1028, 300, 2, False),
    ("g16", 2, 1, 16, 1027, 96, 2, False),
    ("slots", 16, 8, 4, 700, 64, 2, False),
    ("slots_g16", 64, 2, 16, 300, 64, 2, True),
    ("one_query", 3, 2, 4, 2000, 128, 1, False),
    ("one_query_in_place", 3, 2, 4, 2000, 128, 1, True),
    ("long", 1, 2, 4, 70001, 500, 2, False),
    ("long_in_place", 1, 2, 4, 70001, 500, 2, True),
    ("long_one", 1, 2, 4, 70001, 500, 1, False),
    ("ties", 1, 2, 4, 40000, 700, 2, False),
    # more candidates than the many-workgroup selection keeps in registers, its
    # list with positions only and with keys
    ("ties_long", 1, 2, 4, 70001, 500, 2, False),
    ("ties_long_one", 1, 2, 4, 70001, 500, 1, False),
]


@pytest.mark.parametrize("name,B,Hkv,G,n,k,queries,in_place", CASES, ids=[c[0] for c in CASES])
def test_two_queries(name, B, Hkv, G, n, k, queries, in_place):
    print("two queries", name, flush=True)
    dev = device()
    w = dataclasses.replace(synth.WORKLOADS["dual64_s"], name=f"twoq_{name}", batch=B,
                            q_heads=G * Hkv, kv_heads=Hkv, max_ctx=n, ctx_min=max(1, n // 3), k=k,
                            layers=1)
    t = synth.make_layer(w, seed=51, device=dev)
    if B >= 3:
        t["ctx_lens"][0], t["ctx_lens"][1], t["ctx_lens"][2] = 0, k - 1, n
    if name.startswith("ties"):  # almost every score equal
        t["k"][:, :, 100:] = t["k"][:, :, 100:101].clone()
    lens = t["ctx_lens"].cpu().numpy()
    q, K, V = u16(t["q"]), u16(t["k"]), u16(t["v"])
    qs = u16(t["q_sel"]) if queries == 2 else q
    o = orc()
    so = o.shape(B, G * Hkv, Hkv, w.head_dim, n)
    S = [o.score_keys(so, x, K, lens, SCALE, nthreads=8) for x in (q, qs)]
    want = [o.select_topk(so, s, lens, k, nthreads=8) for s in S]
    pred, npred = make_prediction("half", S[0], S[1], lens, k, n, np.random.default_rng(3))

    s = ckv.shape_for(B, G * Hkv, Hkv, n)
    i32 = dict(dtype=torch.int32, device=dev)
    idx_pred, n_pred = torch.from_numpy(pred).to(dev), torch.from_numpy(npred).to(dev)
    kb = torch.zeros((B, Hkv, k, w.head_dim), dtype=torch.bfloat16, device=dev)
    vb = torch.zeros_like(kb)
    ckv.gather_kv(s, t["k"], t["v"], ckv.SRC_DEVICE, idx_pred, n_pred, k, kb, vb)
    idx_true, n_true = torch.full((B, Hkv, k), -9, **i32), torch.full((B, Hkv), -9, **i32)
    idx_next = idx_pred if in_place else torch.full((B, Hkv, k), -9, **i32)
    n_next = n_pred if in_place else torch.full((B, Hkv), -9, **i32)
    hits = torch.full((B, Hkv), -9, **i32)
    out = torch.full((B, G * Hkv, w.head_dim), float("nan"), device=dev)
    ws = ckv.workspace(s, k, ckv.ENTRY_CORRECTED_ATTN)
    ws.fill_(0xA5)
    ckv.corrected_attn(s, t["q"], t["q_sel"] if queries == 2 else None, t["k"], t["ctx_lens"], k,
                       SCALE, t["k"], t["v"], ckv.SRC_DEVICE, idx_pred, n_pred, kb, vb, idx_true,
                       n_true, hits, idx_next, n_next, out, ws)
    torch.cuda.synchronize()
    g_true, g_nt = idx_true.cpu().numpy(), n_true.cpu().numpy()
    check_index_sets(g_true, g_nt, *want[0], S[0], lens)
    check_index_sets(idx_next.cpu().numpy(), n_next.cpu().numpy(), *want[1], S[1], lens)
    for b in range(B):
        for h in range(Hkv):
            both = np.intersect1d(g_true[b, h, :g_nt[b, h]], pred[b, h, :npred[b, h]])
            assert int(hits[b, h]) == len(both), (b, h)
    ref = oracle_attn_over(so, q, K, V, g_true, g_nt, k)
    assert np.abs(out.cpu().numpy() - ref).max() <= ATOL_OUT


@pytest.mark.parametrize("queries", [1, 2])
@pytest.mark.parametrize("n,place", [(4500, "sets"), (70001, "sets"), (4500, "counts"),
                                     (4500, "shifted")])
def test_next_in_the_place_of_results(n, place, queries):
    """The next step's sets written over the call's own sets (idx_next =
    idx_true, n_next = n_true), its counts over the hits, or its sets one unit
    further in the own sets' array: the next step's sets are whole and the
    output is the attention over the own sets."""
    print("next in the place of results", n, place, queries, flush=True)
    dev = device()
    B, Hkv, G, k, d = 2, 2, 4, 96, 128
    w = dataclasses.replace(synth.WORKLOADS["dual64_s"], name=f"twoq_place{n}", batch=B,
                            q_heads=G * Hkv, kv_heads=Hkv, max_ctx=n, ctx_min=n // 3, k=k,
                            layers=1)
    t = synth.make_layer(w, seed=53, device=dev)
    t["ctx_lens"][0] = k - 7  # counts that differ between the units
    lens = t["ctx_lens"].cpu().numpy()
    q, K, V = u16(t["q"]), u16(t["k"]), u16(t["v"])
    o = orc()
    so = o.shape(B, G * Hkv, Hkv, d, n)
    S = [o.score_keys(so, x, K, lens, SCALE, nthreads=8)
         for x in (q, u16(t["q_sel"]) if queries == 2 else q)]
    want = [o.select_topk(so, s, lens, k, nthreads=8) for s in S]
    pred, npred = make_prediction("half", S[0], S[1], lens, k, n, np.random.default_rng(3))

    s = ckv.shape_for(B, G * Hkv, Hkv, n)
    i32 = dict(dtype=torch.int32, device=dev)
    sets = torch.full((B * Hkv + 1, k), -9, **i32)  # one unit more: for the shift
    U = B * Hkv
    idx_true = sets[:U].view(B, Hkv, k)
    n_true, hits, n_next = (torch.full((B, Hkv), -9, **i32) for _ in range(3))
    idx_next = torch.full((B, Hkv, k), -9, **i32)
    if place == "sets":
        idx_next, n_next = idx_true, n_true
    elif place == "counts":
        n_next = hits
    else:
        idx_next = sets[1:].view(B, Hkv, k)
    idx_pred, n_pred = torch.from_numpy(pred).to(dev), torch.from_numpy(npred).to(dev)
    kb = torch.zeros((B, Hkv, k, d), dtype=torch.bfloat16, device=dev)
    vb = torch.zeros_like(kb)
    ckv.gather_kv(s, t["k"], t["v"], ckv.SRC_DEVICE, idx_pred, n_pred, k, kb, vb)
    out = torch.full((B, G * Hkv, d), float("nan"), device=dev)
    ws = ckv.workspace(s, k, ckv.ENTRY_CORRECTED_ATTN)
    ws.fill_(0xA5)
    ckv.corrected_attn(s, t["q"], t["q_sel"] if queries == 2 else None, t["k"], t["ctx_lens"], k,
                       SCALE, t["k"], t["v"], ckv.SRC_DEVICE, idx_pred, n_pred, kb, vb, idx_true,
                       n_true, hits, idx_next, n_next, out, ws)
    torch.cuda.synchronize()
    check_index_sets(idx_next.cpu().numpy(), n_next.cpu().numpy(), *want[1], S[1], lens)
    if place != "counts":
        for b in range(B):
            for h in range(Hkv):
                both = np.intersect1d(want[0][0][b, h, :want[0][1][b, h]], pred[b, h, :npred[b, h]])
                assert int(hits[b, h]) == len(both), (b, h)
    ref = oracle_attn_over(so, q, K, V, *want[0], k)
    assert np.abs(out.cpu().numpy() - ref).max() <= ATOL_OUT


def test_more_units_than_one_launch_selects():
    """The two selections of 2^21 + 8 units of one position: side by side they
    would take more work-items than a launch may have."""
    print("two selections of 2^21 + 8 units", flush=True)
    dev = device()
    U, d = (1 << 21) + 8, 128
    s = ckv.shape_for(1, U, U, 1)
    bf = dict(dtype=torch.bfloat16, device=dev)
    q = torch.ones((1, U, d), **bf)
    keys = torch.ones((1, U, 1, d), **bf)
    vals = (torch.arange(U, device=dev) % 251).to(torch.bfloat16).view(1, U, 1, 1).expand(
        -1, -1, -1, d).contiguous()
    lens = torch.ones(1, dtype=torch.int32, device=dev)
    i32 = lambda v: torch.full((1, U, 1), v, dtype=torch.int32, device=dev)  # noqa: E731
    pred, n_pred = i32(-1), i32(0).view(1, U)
    kb, vb = torch.zeros_like(keys), torch.zeros_like(vals)
    true, nxt = i32(-9), i32(-9)
    n_true, n_next, hits = (i32(-9).view(1, U) for _ in range(3))
    out = torch.full((1, U, d), float("nan"), device=dev)
    ws = ckv.workspace(s, 1, ckv.ENTRY_CORRECTED_ATTN)
    ckv.corrected_attn(s, q, q.clone(), keys, lens, 1, SCALE, keys, vals, ckv.SRC_DEVICE, pred,
                       n_pred, kb, vb, true, n_true, hits, nxt, n_next, out, ws)
    torch.cuda.synchronize()
    for got in (true, nxt, hits):
        assert int(got.abs().max()) == 0
    for got in (n_true, n_next):
        assert int(got.min()) == int(got.max()) == 1
    assert torch.equal(out, vals.view(1, U, d).float())


def test_loop_mixes_one_and_two_queries():
    """Corrected layers of one step share cleared histograms: a layer with one
    query before one with two, at a unit count whose slots hold one query's
    histograms but not two."""
    print("loop of one and two queries", flush=True)
    dev = device()
    B, Hkv, G, n, k, d = 65, 8, 1, 300, 32, 128
    w = dataclasses.replace(synth.WORKLOADS["dual64_s"], name="twoq_loop", batch=B, q_heads=Hkv,
                            kv_heads=Hkv, max_ctx=n, ctx_min=100, k=k, layers=2)
    i32 = dict(dtype=torch.int32, device=dev)
    full = lambda *s: torch.full(s, -9, **i32)  # noqa: E731
    o = orc()
    so = o.shape(B, Hkv, Hkv, d, n)
    layers, want, kept = [], [], []
    for i in range(2):
        t = synth.make_layer(w, seed=71, layer=i, device=dev)
        lens = t["ctx_lens"].cpu().numpy()
        q, qs = u16(t["q"]), u16(t["q_sel"]) if i else u16(t["q"])
        S = [o.score_keys(so, x, u16(t["k"]), lens, SCALE, nthreads=8) for x in (q, qs)]
        want.append([(o.select_topk(so, s, lens, k, nthreads=8), s) for s in S])
        pred, npred = make_prediction("half", S[0], S[1], lens, k, n, np.random.default_rng(i))
        layers.append({"q_att": t["q"], "q_sel": t["q_sel"] if i else None, "k_score": t["k"],
                       "k_src": t["k"], "v_src": t["v"], "idx_prev": torch.from_numpy(pred).to(dev),
                       "n_sel_prev": torch.from_numpy(npred).to(dev), "idx_next": full(B, Hkv, k),
                       "n_sel_next": full(B, Hkv), "idx_true": full(B, Hkv, k),
                       "n_true": full(B, Hkv), "hits": full(B, Hkv),
                       "out": torch.zeros((B, Hkv, d), device=dev)})
        kept.append(t)
    s = ckv.shape_for(B, Hkv, Hkv, n)
    ws = ckv.workspace(s, k, ckv.ENTRY_CORRECTED_ATTN)
    ws.fill_(0xA5)
    bufs = [torch.zeros((B, Hkv, k, d), dtype=torch.bfloat16, device=dev) for _ in range(4)]
    pipe, copy = ckv.Pipeline(), torch.cuda.Stream()
    torch.cuda.synchronize()
    pipe.prime(s, k, layers, ckv.SRC_DEVICE, bufs[:2], bufs[2:], copy)
    pipe.step(s, layers, kept[0]["ctx_lens"], k, SCALE, ckv.SRC_DEVICE, bufs[:2], bufs[2:], ws,
              None, copy)
    torch.cuda.synchronize()
    pipe.close()
    for l, ((true, s1), (nxt, s2)) in zip(layers, want):
        check_index_sets(l["idx_true"].cpu().numpy(), l["n_true"].cpu().numpy(), *true, s1, lens)
        check_index_sets(l["idx_next"].cpu().numpy(), l["n_sel_next"].cpu().numpy(), *nxt, s2, lens)
