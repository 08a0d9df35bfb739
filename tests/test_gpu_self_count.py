"""Selections that count their own first digit (MI355X only): select_topk of
contexts up to 65536 positions, and same-step and pipelined calls of few units
and up to 24576.  Sizes at the edges of the 8192-position chunks and of the
32768 positions held in registers; crowded scores overflow a wave's candidate
segment.  The sets must be the oracle's on the GPU's own fp32 scores, exactly.
"""
from __future__ import annotations

import dataclasses

import numpy as np
import pytest
import torch

import paper_2607_26475_amd as ckv
import synth
from helpers import ATOL_OUT, SCALE, Run, device, oracle_attn_over, orc, u16

pytestmark = pytest.mark.gpu

CASES = [(1, 1), (64, 5), (8191, 600), (8192, 512), (8193, 7), (16385, 2048), (24576, 1000),
         (24577, 1000), (32768, 300), (32769, 4000), (40961, 20000), (65536, 2048), (65536, 65535)]


@pytest.mark.parametrize("crowded", [False, True], ids=["spread", "crowded"])
@pytest.mark.parametrize("n,k", CASES)
def test_self_counting_selection(n, k, crowded):
    print("self-counting selection", n, k, crowded, flush=True)
    dev = device()
    B, Hkv, G, d = 2, 1, 2, 128
    w = dataclasses.replace(synth.WORKLOADS["dual64_s"], name=f"selfcount{n}", batch=B,
                            q_heads=Hkv * G, kv_heads=Hkv, max_ctx=n, ctx_min=n, k=k, layers=1)
    t = synth.make_layer(w, seed=61, device=dev)
    lens = torch.tensor([n, max(0, n - 37)], dtype=torch.int32, device=dev)
    if crowded:  # a few distinct scores
        t["k"].copy_(t["k"][:, :, torch.arange(n, device=dev) % min(n, 5)].clone())
    s = ckv.shape_for(B, Hkv * G, Hkv, n)
    scores = torch.empty((B, Hkv, n), device=dev)
    ckv.score_keys(s, t["q_sel"], t["k"], lens, SCALE, scores)
    i32 = dict(dtype=torch.int32, device=dev)
    idx, nsel = torch.full((B, Hkv, k), -9, **i32), torch.full((B, Hkv), -9, **i32)
    ws = ckv.workspace(s, k, ckv.ENTRY_SELECT_TOPK)
    ws.fill_(0xA5)
    ckv.select_topk(s, scores, lens, k, idx, nsel, ws)
    run, pipe = Run(w, lens, dev), Run(w, lens, dev)
    run.same_step(t["q"], t["q_sel"], t["k"], t["k"], t["v"], ckv.SRC_DEVICE)
    pipe.in_place(t["q"], t["q_sel"], t["k"], t["k"], t["v"], ckv.SRC_DEVICE, run.idx, run.n_sel)
    torch.cuda.synchronize()
    o = orc()
    so = o.shape(B, Hkv * G, Hkv, d, n)
    ln = lens.cpu().numpy()
    want = o.select_topk(so, scores.cpu().numpy().astype(np.float64), ln, k, nthreads=8)
    for got in ((idx, nsel), (run.idx, run.n_sel), (pipe.idx, pipe.n_sel)):
        np.testing.assert_array_equal(got[1].cpu().numpy(), want[1])
        np.testing.assert_array_equal(got[0].cpu().numpy(), want[0])
    ref = oracle_attn_over(so, u16(t["q"]), u16(t["k"]), u16(t["v"]), *want, k)
    assert np.abs(run.out.cpu().numpy() - ref).max() <= ATOL_OUT
    assert np.abs(pipe.out.cpu().numpy() - ref).max() <= ATOL_OUT
