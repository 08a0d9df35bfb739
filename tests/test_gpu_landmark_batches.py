"""Chunk landmarks at the edges of the batches of rows a thread loads (MI355X
only): every batch of 1 to 16 rows, chunks of several rounds, chunks that divide
by a power of two and others, partial last chunks, bit for bit against the
oracle."""
from __future__ import annotations

import dataclasses

import numpy as np
import pytest
import torch

import paper_2607_26475_amd as ckv
import synth
from helpers import device, orc, u16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chunk", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16, 17, 20, 32, 33, 700])
def test_landmark_batches(chunk):
    print("landmark batches", chunk, flush=True)
    dev = device()
    B, Hkv, n, d = 3, 2, 601, 128
    w = dataclasses.replace(synth.WORKLOADS["dual64_s"], name="lmbatch", batch=B, q_heads=8,
                            kv_heads=Hkv, max_ctx=n, ctx_min=n, k=64)
    t = synth.make_layer(w, seed=chunk, device=dev)
    lens = np.array([n, 0, 256 + chunk], np.int32).clip(0, n)
    cmax = -(-n // chunk)
    out = torch.full((B, Hkv, cmax, d), float("nan"), dtype=torch.bfloat16, device=dev)
    ckv.chunk_landmarks(ckv.shape_for(B, 8, Hkv, n), chunk, t["k"], torch.from_numpy(lens).to(dev),
                        out)
    torch.cuda.synchronize()
    got = u16(out)
    o = orc()
    want = o.chunk_landmarks(o.shape(B, 8, Hkv, d, n), chunk, u16(t["k"]), lens)
    for b in range(B):
        nc = -(-int(lens[b]) // chunk)
        np.testing.assert_array_equal(got[b, :, :nc], want[b, :, :nc])
        assert np.all(np.isnan(out[b, :, nc:].float().cpu().numpy())), "later landmarks written"
