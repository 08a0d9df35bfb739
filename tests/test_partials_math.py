"""Which batches get per-workgroup histogram slots, and how many a unit has, by
brute force (no GPU).

The library's own functions, compiled for the host.  slots_fit promises from
the stored shape alone that the units of a full batch meet at most `slots` of
the even ranges.  With slots the ranges are at least min_range_groups long, so
that no unit of any batch meets more than the selection reads; slots must be
unique and below units + nwg.
"""
from __future__ import annotations

import numpy as np
import pytest

from native_ranges import lib, pair

CASES = [(1, 1, 1), (2, 5, 3), (128, 1024, 512), (128, 94, 512), (256, 47, 512), (16, 7, 100),
         (3, 1000, 7), (64, 4096, 1024), (5, 3, 15), (16, 1024, 256), (24, 1024, 256),
         (36, 188, 256), (40, 188, 256), (520, 10, 256)]


@pytest.mark.parametrize("U,gu,nwg", CASES)
def test_slots_fit_full_batches(U, gu, nwg):
    so = lib()
    nwg = min(nwg, U * gu)  # the grid never has more workgroups than groups
    R = so.t_range_groups(U * gu, nwg, 1)
    most = max(pair(so.t_unit_ranges, u * gu, gu, R)[1] for u in range(U))
    for slots in range(2, 40):
        if so.t_slots_fit(gu, U, nwg, slots):
            assert most <= slots
    # the promise is within two of what the units meet
    assert so.t_slots_fit(gu, U, nwg, most + 2 + (gu * U) % nwg)


@pytest.mark.parametrize("U,gu,nwg", CASES)
def test_slots_of_ragged_batches(U, gu, nwg):
    so = lib()
    nwg, most = min(nwg, U * gu), so.t_max_partials()
    rng = np.random.default_rng(U * 7 + gu)
    for trial in range(8):
        vg = rng.integers(0, gu + 1, size=U) if trial else np.eye(1, U, U // 2, dtype=int)[0] * gu
        R = so.t_range_groups(int(vg.sum()), nwg, so.t_min_range_groups(gu, most))
        seen, base = set(), 0
        for u, g in enumerate(vg.tolist()):
            first, count = pair(so.t_unit_ranges, base, g, R)
            assert count <= most, (u, g)
            for s in range(u + first, u + first + count):
                assert s not in seen and s < U + nwg
                seen.add(s)
            base += g


@pytest.mark.parametrize("units,fit8,fit16", [(16, 0, 0), (18, 0, 1), (24, 0, 1), (36, 0, 1),
                                              (37, 1, 1), (40, 1, 1)])
def test_slots_edge(units, fit8, fit16):
    """256 workgroups and 32 Ki positions: 8 slots from 37 units, 16 from 18."""
    so = lib()
    gu = so.t_groups_of(32768)
    assert so.t_slots_fit(gu, units, 256, 8) == fit8
    assert so.t_slots_fit(gu, units, 256, 16) == fit16
