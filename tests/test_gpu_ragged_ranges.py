"""Scoring ranges over the positions below each request's length (MI355X only).

Ranges are cut from the valid groups of the whole batch, so the cases put
empty requests between others, one long request among empty ones (where the
least range length sets the split), a request per unit for more than 64
requests (the length scan takes several steps), and nothing at all, through
score_keys, the same-step call (one launch, slots, added histograms) and the
pipelined call, against the oracle.
"""
from __future__ import annotations

import dataclasses

import numpy as np
import pytest
import torch

import paper_2607_26475_amd as ckv
import synth
from helpers import (ATOL_OUT, SCALE, Run, check_index_sets, check_scores, device,
                     oracle_attn_over, orc, u16)

pytestmark = pytest.mark.gpu


def _few_long(B, n, short):
    rng = np.random.default_rng(B)
    lens = rng.integers(0, short, size=B)
    lens[[3, B - 2]] = n
    return [int(x) for x in lens]


CASES = [  # name, B, Hq, Hkv, stored rows, k, lengths
    ("one_full", 16, 32, 8, 6000, 512, [6000] + [0] * 15),
    ("one_full_last", 16, 32, 8, 6000, 512, [0] * 15 + [6000]),
    ("gaps", 16, 32, 8, 3001, 512, [0, 1, 33, 3001, 0, 0, 32, 3000, 1, 0, 31, 2, 0, 700, 64, 0]),
    ("many_requests", 130, 4, 1, 1500, 256, _few_long(130, 1500, 900)),
    ("many_long", 70, 4, 1, 66000, 128, _few_long(70, 66000, 300)),
    ("all_empty", 16, 32, 8, 3000, 512, [0] * 16),
    # more slots per unit than one round of the selection's loads takes
    ("many_slots", 6, 32, 8, 20000, 256, [20000, 19000, 0, 20000, 7000, 20000]),
    ("many_slots_long", 3, 32, 8, 26000, 600, [26000, 25000, 26000]),
]


@pytest.mark.parametrize("name,B,Hq,Hkv,n,k,lens", CASES, ids=[c[0] for c in CASES])
def test_ragged_ranges(name, B, Hq, Hkv, n, k, lens):
    print("ragged ranges", name, flush=True)
    dev = device()
    w = dataclasses.replace(synth.WORKLOADS["dual64_s"], name=f"ragged_{name}", batch=B,
                            q_heads=Hq, kv_heads=Hkv, max_ctx=n, ctx_min=n, k=k, layers=1)
    t = synth.make_layer(w, seed=41, device=dev)
    dl = torch.tensor(lens, dtype=torch.int32, device=dev)
    ln = np.array(lens)
    q, qs, K, V = u16(t["q"]), u16(t["q_sel"]), u16(t["k"]), u16(t["v"])
    o = orc()
    so = o.shape(B, Hq, Hkv, w.head_dim, n)
    S = o.score_keys(so, qs, K, ln, SCALE, nthreads=8)
    r_idx, r_nsel = o.select_topk(so, S, ln, k, nthreads=8)

    s = ckv.shape_for(B, Hq, Hkv, n)
    scores = torch.full((B, Hkv, n), float("nan"), device=dev)
    ckv.score_keys(s, t["q_sel"], t["k"], dl, SCALE, scores)
    torch.cuda.synchronize()
    check_scores(scores.cpu().numpy(), S, qs, K, ln, Hq // Hkv)

    run = Run(w, dl, dev)
    run.same_step(t["q"], t["q_sel"], t["k"], t["k"], t["v"], ckv.SRC_DEVICE)
    g_idx, g_nsel, g_out = run.host()
    check_index_sets(g_idx, g_nsel, r_idx, r_nsel, S, ln)
    ref = oracle_attn_over(so, q, K, V, g_idx, g_nsel, k)
    assert np.abs(g_out - ref).max() <= ATOL_OUT

    pipe = Run(w, dl, dev)
    pipe.in_place(t["q"], t["q_sel"], t["k"], t["k"], t["v"], ckv.SRC_DEVICE, run.idx, run.n_sel)
    p_idx, p_nsel, p_out = pipe.host()
    np.testing.assert_array_equal(p_idx, g_idx)
    np.testing.assert_array_equal(p_nsel, g_nsel)
    assert np.abs(p_out - ref).max() <= ATOL_OUT
