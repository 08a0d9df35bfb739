"""select_topk past 65536 positions (MI355X only): the filter's tiles of 16384
positions, the finish's candidates in registers and in its list, and the
ordered output from LDS and memory bitmaps whose word counts are not multiples
of 4 or 32, sparse and dense, and on both sides of the selection of a position in
16 that tells them apart.  Exactly the oracle's sets on the same scores."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2607_26475_amd as ckv
from helpers import device, orc

pytestmark = pytest.mark.gpu

CASES = [(65537, 1), (70003, 30000), (81920, 4096), (81921, 81000), (131072, 2048),
         (1048575, 9000), (1048643, 40000), (65600, 4099), (65600, 4100), (65600, 4102),
         (1048545, 400000), (1048643, 700000)]


@pytest.mark.parametrize("n,k", CASES)
def test_long_select(n, k):
    print("long select", n, k, flush=True)
    dev = device()
    B = 2
    rng = np.random.default_rng(n + k)
    sc = rng.standard_normal((B, 1, n)).astype(np.float32)
    sc[1, 0, ::3] = 1.5  # a third of the scores tied
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
    want = o.select_topk(o.shape(B, 4, 1, 128, n), sc.astype(np.float64), lens, k, nthreads=8)
    np.testing.assert_array_equal(nsel.cpu().numpy(), want[1])
    np.testing.assert_array_equal(idx.cpu().numpy(), want[0])
