"""Adaptive key reconstruction (Sec. 5.3) against the oracle (MI355X only).

ckv_reconstruct_keys must rebuild every requested key bit for bit as the
oracle does (fp64 sum over the rank in ascending order, rounded once to bf16),
leave untouched the slots it must not write, and ckv_corrected_attn_lowrank
must attend over the prefetched keys of the hits and the rebuilt keys of the
misses, with every value fetched.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2607_26475_amd as ckv
import synth
from helpers import (ATOL_OUT, SCALE, check_index_sets, device, make_prediction,
                     oracle_lowrank_buffers, orc, u16)

pytestmark = pytest.mark.gpu

FILL = 0x7777


def _log(*a):
    print(*a, flush=True)


def _requests(w, lens, counts, rng, invalid=False):
    """Ascending distinct rows below n_b per unit, -1 padded, and the counts
    to pass (which may be negative or above k: the library clamps them).
    With invalid, a few entries below the count point outside [0, max_ctx)."""
    B, Hkv, k = w.batch, w.kv_heads, w.k
    idx = np.full((B, Hkv, k), -1, np.int32)
    cnt = np.zeros((B, Hkv), np.int32)
    for b in range(B):
        n = int(lens[b])
        for h in range(Hkv):
            c = counts[(b * Hkv + h) % len(counts)]
            m = max(0, min(c, k, n))
            idx[b, h, :m] = np.sort(rng.choice(n, size=m, replace=False))
            cnt[b, h] = c
            if invalid and m >= 3:
                idx[b, h, 0] = -1
                idx[b, h, m // 2] = w.max_ctx
                idx[b, h, m - 1] = w.max_ctx + 1000
    return idx, cnt


@pytest.mark.parametrize("wl,rank", [("tiny", 1), ("tiny", 7), ("dual64_s", 64),
                                     ("llama8b_s", 160)])
def test_reconstruct_keys_bit_exact(wl, rank):
    _log("reconstruct", wl, rank)
    dev = device()
    w = synth.WORKLOADS[wl]
    B, Hq, Hkv, d, k, n = w.batch, w.q_heads, w.kv_heads, w.head_dim, w.k, w.max_ctx
    t = synth.make_layer(w, seed=2, device=dev)
    lens = t["ctx_lens"].cpu().numpy()
    u_fac, w_fac = synth.low_rank_factors(w, rank, seed=2, device=dev)
    U, W = u16(u_fac), u16(w_fac)
    rng = np.random.default_rng(rank)
    idx, cnt = _requests(w, lens, [k, 0, k // 3, -5, k + 9, 1], rng)
    s = ckv.shape_for(B, Hq, Hkv, n)
    k_dst = torch.full((B, Hkv, k, d), FILL, dtype=torch.int16, device=dev)
    ckv.reconstruct_keys(s, rank, u_fac, w_fac, torch.from_numpy(idx).to(dev),
                         torch.from_numpy(cnt).to(dev), k, k_dst)
    torch.cuda.synchronize()
    got = k_dst.cpu().numpy().view(np.uint16)
    o = orc()
    so = o.shape(B, Hq, Hkv, d, n)
    want = o.reconstruct_keys(so, rank, U, W, idx, cnt, k, fill=FILL)
    bad = np.argwhere(got != want)
    assert len(bad) == 0, (len(bad), bad[:4])


def test_reconstruct_keys_skips_rows_out_of_range():
    _log("reconstruct invalid rows")
    dev = device()
    w = synth.WORKLOADS["dual64_s"]
    B, Hq, Hkv, d, k, n = w.batch, w.q_heads, w.kv_heads, w.head_dim, w.k, w.max_ctx
    rank = 16
    lens = synth.make_layer(w, seed=4, device="cpu")["ctx_lens"].numpy()
    u_fac, w_fac = synth.low_rank_factors(w, rank, seed=4, device=dev)
    idx, cnt = _requests(w, lens, [k, 100, 37], np.random.default_rng(1), invalid=True)
    s = ckv.shape_for(B, Hq, Hkv, n)
    k_dst = torch.full((B, Hkv, k, d), FILL, dtype=torch.int16, device=dev)
    ckv.reconstruct_keys(s, rank, u_fac, w_fac, torch.from_numpy(idx).to(dev),
                         torch.from_numpy(cnt).to(dev), k, k_dst)
    torch.cuda.synchronize()
    got = k_dst.cpu().numpy().view(np.uint16)
    # the oracle rebuilds only valid rows: invalid ones are asked as row 0
    bad = (idx < 0) | (idx >= n)
    o = orc()
    want = o.reconstruct_keys(o.shape(B, Hq, Hkv, d, n), rank, u16(u_fac), u16(w_fac),
                              np.where(bad, 0, idx), cnt, k, fill=FILL)
    want[bad] = FILL
    np.testing.assert_array_equal(got, want)


LOWRANK_CASES = [
    ("dual64_s", "speculative", ckv.SRC_HOST_PINNED, 32),
    ("dual64_s", "disjoint", ckv.SRC_DEVICE, 160),
    ("llama8b_s", "half", ckv.SRC_HOST_PINNED, 64),
    ("tiny", "exact", ckv.SRC_DEVICE, 8),
    ("tiny", "empty", ckv.SRC_HOST_PINNED, 8),
    # on both sides of the ranks that one thread sums
    ("dual64_s", "half", ckv.SRC_DEVICE, 3),
    ("dual64_s", "disjoint", ckv.SRC_HOST_PINNED, 8),
    ("dual64_s", "disjoint", ckv.SRC_DEVICE, 9),
]


@pytest.mark.parametrize("wl,kind,src_kind,rank", LOWRANK_CASES)
def test_corrected_attn_lowrank(wl, kind, src_kind, rank):
    _log("corrected lowrank", wl, kind, src_kind, rank)
    dev = device()
    w = synth.WORKLOADS[wl]
    B, Hq, Hkv, d, k, n = w.batch, w.q_heads, w.kv_heads, w.head_dim, w.k, w.max_ctx
    t = synth.make_layer(w, seed=6, device=dev)
    lens = t["ctx_lens"]
    lens_h = lens.cpu().numpy()
    q_att, q_sel, K, V = u16(t["q"]), u16(t["q_sel"]), u16(t["k"]), u16(t["v"])
    u_fac, w_fac = synth.low_rank_factors(w, rank, seed=6, device=dev)
    o = orc()
    so = o.shape(B, Hq, Hkv, d, n)
    S_att = o.score_keys(so, q_att, K, lens_h, SCALE, nthreads=8)
    S_sel = o.score_keys(so, q_sel, K, lens_h, SCALE, nthreads=8)
    pred, npred = make_prediction(kind, S_att, S_sel, lens_h, k, n, np.random.default_rng(9))

    if src_kind == ckv.SRC_HOST_PINNED:
        kv = synth.host_kv(t["k"], t["v"])
        k_src, v_src, stride = kv.data_ptr(), kv.data_ptr() + 2 * d, 2 * d
    else:
        k_src, v_src, stride = t["k"], t["v"], d
    s = ckv.shape_for(B, Hq, Hkv, n, kv_row_stride=stride)
    idx_pred = torch.from_numpy(pred).to(dev)
    n_pred = torch.from_numpy(npred).to(dev)
    k_buf = torch.zeros((B, Hkv, k, d), dtype=torch.bfloat16, device=dev)
    v_buf = torch.zeros_like(k_buf)
    ckv.gather_kv(s, k_src, v_src, src_kind, idx_pred, n_pred, k, k_buf, v_buf)  # the prefetch
    k_buf2, v_buf2 = k_buf.clone(), v_buf.clone()
    i32 = dict(dtype=torch.int32, device=dev)
    idx_true, idx_next = torch.full((B, Hkv, k), -9, **i32), torch.full((B, Hkv, k), -9, **i32)
    n_true, n_next, hits = (torch.full((B, Hkv), -9, **i32) for _ in range(3))
    out = torch.full((B, Hq, d), float("nan"), device=dev)
    ws = ckv.workspace(s, k, ckv.ENTRY_CORRECTED_ATTN)
    ws.fill_(0xA5)
    # keys are rebuilt: no key source is passed
    ckv.corrected_attn_lowrank(s, t["q"], t["q_sel"], t["k"], lens, k, SCALE, None, v_src,
                               src_kind, rank, u_fac, w_fac, idx_pred, n_pred, k_buf, v_buf,
                               idx_true, n_true, hits, idx_next, n_next, out, ws)
    # the same layer fetching its misses whole, for comparison
    out2 = torch.full_like(out, float("nan"))
    idx_t2, n_t2, hits2 = torch.empty_like(idx_true), torch.empty_like(n_true), torch.empty_like(hits)
    ckv.corrected_attn(s, t["q"], t["q_sel"], t["k"], lens, k, SCALE, k_src, v_src, src_kind,
                       idx_pred, n_pred, k_buf2, v_buf2, idx_t2, n_t2, hits2,
                       torch.empty_like(idx_next), torch.empty_like(n_next), out2, ws)
    torch.cuda.synchronize()
    g_true, g_nt = idx_true.cpu().numpy(), n_true.cpu().numpy()
    g_next, g_nn = idx_next.cpu().numpy(), n_next.cpu().numpy()
    g_hits, g_out = hits.cpu().numpy(), out.cpu().numpy()

    r_true, r_nt = o.select_topk(so, S_att, lens_h, k, nthreads=8)
    check_index_sets(g_true, g_nt, r_true, r_nt, S_att, lens_h)
    r_next, r_nn = o.select_topk(so, S_sel, lens_h, k, nthreads=8)
    check_index_sets(g_next, g_nn, r_next, r_nn, S_sel, lens_h)
    np.testing.assert_array_equal(g_true, idx_t2.cpu().numpy())
    np.testing.assert_array_equal(g_hits, hits2.cpu().numpy())
    total = found = 0
    for b in range(B):
        for h in range(Hkv):
            want = len(np.intersect1d(g_true[b, h, :g_nt[b, h]], pred[b, h, :npred[b, h]]))
            assert g_hits[b, h] == want, (b, h, g_hits[b, h], want)
            total += g_nt[b, h]
            found += want
    kb, vb = oracle_lowrank_buffers(so, K, V, rank, u16(u_fac), u16(w_fac), g_true, g_nt,
                                    pred, npred, k)
    ref = o.sparse_decode_attn(so, q_att, kb, vb, g_nt, k, SCALE, nthreads=8)
    err = np.abs(g_out - ref).max() if g_out.size else 0.0
    _log(f"  hit rate {found / max(total, 1):.3f}, max abs err {err:.2e}")
    assert err <= ATOL_OUT
    if found == total:  # nothing rebuilt: the same buffer, the same kernels, the same bits
        np.testing.assert_array_equal(g_out, out2.cpu().numpy())
    # the buffer holds each selected row's (key, value) pair: rebuilt key for misses
    kbg = k_buf.cpu().view(torch.int16).numpy()
    vbg = v_buf.cpu().view(torch.int16).numpy()
    for b in range(B):
        for h in range(Hkv):
            pairs = {kbg[b, h, s_].tobytes() + vbg[b, h, s_].tobytes() for s_ in range(k)}
            for i in range(int(g_nt[b, h])):
                key = kb[b, h, i].view(np.int16).tobytes() + vb[b, h, i].view(np.int16).tobytes()
                assert key in pairs, (b, h, i, int(g_true[b, h, i]))
