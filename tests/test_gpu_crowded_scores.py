"""Crowded scores (MI355X only): more of a wave's positions in the cut's
first-digit bin (a quarter of an octave of the score) than its candidate
segment holds, so that the selection counts the second digit over all
positions and lists the bin of both digits; and, where ties fill that too,
looks candidates up among all positions.  Sets exactly the oracle's on the
GPU's own fp32 scores.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2607_26475_amd as ckv
from helpers import ATOL_OUT, SCALE, device, oracle_attn_over, orc, u16

pytestmark = pytest.mark.gpu

D = 128


def _scores(kind, rng, shape):
    x = rng.standard_normal(shape)
    s = {"offset": 10 + x, "negative": -10 + x, "narrow": 1 + 0.01 * rng.random(shape),
         "tiny": 1e-39 * (1 + rng.random(shape)),  # denormal
         "half_tied": np.where(rng.random(shape) < 0.5, 12.0, 10 + x),
         "coarse": np.round(20 + 2 * x) / 2,        # some 20 distinct scores
         "signs": np.where(x > 0, 0.0, -0.0)}[kind].astype(np.float32)
    flat = s.reshape(-1)
    if kind == "offset":
        flat[rng.integers(0, flat.size, 40)] = np.inf
        flat[rng.integers(0, flat.size, 40)] = -np.inf
    return s


@pytest.mark.parametrize("kind", ["offset", "negative", "narrow", "tiny", "half_tied", "coarse",
                                  "signs"])
@pytest.mark.parametrize("n,k", [(8193, 100), (24576, 6000), (32769, 2048), (65536, 1), (65536, 2048),
                                 (65521, 40000)])
def test_crowded_select(n, k, kind):
    print("crowded select", n, k, kind, flush=True)
    dev = device()
    B = 2
    sc = _scores(kind, np.random.default_rng(n + k), (B, 1, n))
    lens = np.array([n, n - 29], np.int32)
    s = ckv.shape_for(B, 4, 1, n)
    idx = torch.full((B, 1, k), -9, dtype=torch.int32, device=dev)
    nsel = torch.full((B, 1), -9, dtype=torch.int32, device=dev)
    ws = ckv.workspace(s, k, ckv.ENTRY_SELECT_TOPK)
    ws.fill_(0xA5)
    ckv.select_topk(s, torch.from_numpy(sc).to(dev), torch.from_numpy(lens).to(dev), k, idx, nsel,
                    ws)
    torch.cuda.synchronize()
    o = orc()
    want = o.select_topk(o.shape(B, 4, 1, D, n), sc.astype(np.float64), lens, k, nthreads=8)
    np.testing.assert_array_equal(nsel.cpu().numpy(), want[1])
    np.testing.assert_array_equal(idx.cpu().numpy(), want[0])


@pytest.mark.parametrize("B,H,n,k", [(1, 2, 20000, 512), (2, 4, 40000, 700), (8, 8, 40001, 512),
                                     (8, 8, 65536, 600)])
def test_crowded_calls(B, H, n, k):
    """Keys along the group's query: scores of mean 10 and spread 1, through the
    same-step call (one launch at 64 units), the pipelined one, and the loop
    whose selections run in the next layer's launch."""
    print("crowded calls", B, H, n, k, flush=True)
    dev = device()
    G = 2
    g = torch.Generator(device=dev)
    g.manual_seed(n + k)
    rn = lambda *s: torch.randn(s, generator=g, device=dev)  # noqa: E731
    q0 = rn(B, H, 1, D)
    q = (q0 + 0.1 * rn(B, H, G, D)).reshape(B, H * G, D).bfloat16()
    K = (rn(B, H, n, D) + 10 * q0 / q0.norm(dim=-1, keepdim=True)).bfloat16()
    V = rn(B, H, n, D).bfloat16()
    lens = torch.tensor([n - 31 * b for b in range(B)], dtype=torch.int32, device=dev)
    s = ckv.shape_for(B, H * G, H, n)
    scores = torch.empty((B, H, n), device=dev)
    ckv.score_keys(s, q, K, lens, SCALE, scores)
    o, ln = orc(), lens.cpu().numpy()
    so = o.shape(B, H * G, H, D, n)
    sc = scores.cpu().numpy().astype(np.float64)
    cut = np.sort(sc[0, 0, :n])[-k]
    assert np.mean(sc[0, 0, :n] > cut - 1) > 0.05  # a crowded cut
    want = o.select_topk(so, sc, ln, k, nthreads=8)
    full = lambda *x: torch.full(x, -9, dtype=torch.int32, device=dev)  # noqa: E731
    d_idx, d_n = torch.from_numpy(want[0]).to(dev), torch.from_numpy(want[1]).to(dev)
    outs = [torch.zeros((B, H * G, D), device=dev) for _ in range(4)]
    sets = [(full(B, H, k), full(B, H)) for _ in range(4)]
    ws = ckv.workspace(s, k, ckv.ENTRY_DECODE_STEP)
    ws.fill_(0xA5)
    ckv.critical_kv_attn(s, q, None, K, lens, k, SCALE, K, V, ckv.SRC_DEVICE, None, None, None,
                         *sets[0], outs[0], ws)
    ckv.critical_kv_attn(s, q, None, K, lens, k, SCALE, K, V, ckv.SRC_DEVICE, None, None, d_n,
                         *sets[1], outs[1], ws, idx_in=d_idx)
    layers = [{"q_att": q, "q_sel": None, "k_score": K, "k_src": K, "v_src": V, "idx_prev": d_idx,
               "n_sel_prev": d_n, "idx_next": sets[i][0], "n_sel_next": sets[i][1],
               "out": outs[i]} for i in (2, 3)]
    pipe = ckv.Pipeline()
    pipe.step(s, layers, lens, k, SCALE, ckv.SRC_DEVICE, None, None, ws, None, 0)
    torch.cuda.synchronize()
    pipe.close()
    ref = oracle_attn_over(so, u16(q), u16(K), u16(V), *want, k)
    for (idx, n_sel), out in zip(sets, outs):
        np.testing.assert_array_equal(n_sel.cpu().numpy(), want[1])
        np.testing.assert_array_equal(idx.cpu().numpy(), want[0])
        assert np.abs(out.cpu().numpy() - ref).max() <= ATOL_OUT
