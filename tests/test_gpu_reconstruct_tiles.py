"""Rebuilt keys at the edges of the matrix tiles and of the ranks summed per
thread instead (up to 8) (MI355X only): row counts
around 32, ranks around the 4 of a product and the 64 staged at a time, odd
ranks (rows that do not start on 16 bytes), bit for bit against the oracle's
ordered fp64 sums, with factors whose magnitudes spread over 2^40 so that the
order and the rounding of every addition show.
"""
from __future__ import annotations

import dataclasses

import numpy as np
import pytest
import torch

import paper_2607_26475_amd as ckv
import synth
from helpers import device, orc, u16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rank,counts", [(1, [70, 33]), (3, [1, 31]), (4, [32, 33]),
                                         (8, [33, 70]), (9, [64, 33]), (63, [64, 65]),
                                         (64, [70, 0]), (65, [31, 32]), (72, [33, 70]),
                                         (130, [70, 15]), (200, [17, 64])])
def test_reconstruct_tiles(rank, counts):
    print("reconstruct tiles", rank, counts, flush=True)
    dev = device()
    k, n, B, Hkv, d = 70, 90, 1, 2, 128
    w = dataclasses.replace(synth.WORKLOADS["dual64_s"], name="rectiles", batch=B, q_heads=8,
                            kv_heads=Hkv, max_ctx=n, ctx_min=n, k=k)
    u_fac, w_fac = synth.low_rank_factors(w, rank, seed=rank, device=dev)
    rng = np.random.default_rng(rank)
    spread = torch.from_numpy(2.0 ** rng.integers(-20, 21, size=rank)).to(dev)
    u_fac = (u_fac.double() * spread).to(torch.bfloat16)
    idx = np.full((B, Hkv, k), -1, np.int32)
    for h in range(Hkv):
        idx[0, h, :counts[h]] = np.sort(rng.choice(n, size=counts[h], replace=False))
    cnt = np.array([counts], np.int32)
    k_dst = torch.full((B, Hkv, k, d), 0x7E55, dtype=torch.int16, device=dev)
    ckv.reconstruct_keys(ckv.shape_for(B, 8, Hkv, n), rank, u_fac, w_fac,
                         torch.from_numpy(idx).to(dev), torch.from_numpy(cnt).to(dev), k, k_dst)
    torch.cuda.synchronize()
    o = orc()
    want = o.reconstruct_keys(o.shape(B, 8, Hkv, d, n), rank, u16(u_fac), u16(w_fac), idx, cnt, k,
                              fill=0x7E55)
    np.testing.assert_array_equal(k_dst.cpu().numpy().view(np.uint16), want)
