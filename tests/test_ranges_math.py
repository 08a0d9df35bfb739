"""The scoring pass's ranges over valid groups, by brute force (no GPU).

The library's own functions, compiled for the host: items (requests with
``mult`` units each) have vg groups per unit; groups are numbered unit-major
and cut into ranges of R = range_groups(total, nwg, least).  Every group must
lie in exactly one of the nwg ranges, the workgroups that meet a unit must be
the ones that unit_ranges names, slot unit + workgroup must be unique and below
U + nwg, and with the least range of a slot budget no unit may meet more ranges
than it.  The same where ranges count the stored groups of every unit and a
unit's valid ones are its first.
"""
from __future__ import annotations

import numpy as np
import pytest

from native_ranges import lib, pair


@pytest.mark.parametrize("stored", [False, True], ids=["valid", "stored"])
@pytest.mark.parametrize("items,mult,gu,nwg,slots", [
    (1, 1, 1, 1, 8), (16, 8, 188, 256, 8), (130, 1, 47, 256, 8), (70, 2, 300, 512, 8),
    (5, 3, 15, 64, 8), (16, 8, 1024, 512, 16), (3, 4, 2048, 256, 8), (9, 1, 8, 100, 2)])
def test_ranges(items, mult, gu, nwg, slots, stored):
    so = lib()
    rng = np.random.default_rng(items * 31 + gu)
    for trial in range(12):
        vg = rng.integers(0, gu + 1, size=items)
        if trial == 0:
            vg[:] = gu
        elif trial == 1:
            vg[:] = 0
        elif trial == 2:
            vg[:] = 0
            vg[rng.integers(items)] = gu
        units = np.repeat(vg, mult)
        counted = np.full_like(units, gu) if stored else units
        total = int(counted.sum())
        for least in (1, so.t_added_min_range(gu), so.t_min_range_groups(gu, slots)):
            R = so.t_range_groups(total, nwg, least)
            ranges = [pair(so.t_range_of, w, R, total) for w in range(nwg)]
            assert sum(b - a for a, b in ranges) == total
            assert all(a == b0 for (_, b0), (a, _) in zip(ranges, ranges[1:]))
            seen, base = set(), 0
            for u, (g, c) in enumerate(zip(units.tolist(), counted.tolist())):
                first, count = pair(so.t_unit_ranges, base, g, R)
                meets = [w for w, (a, b) in enumerate(ranges) if a < base + g and b > base]
                if g:
                    assert meets == list(range(first, first + count))
                    for w in meets:
                        assert u + w not in seen and u + w < len(units) + nwg
                        seen.add(u + w)
                else:  # no range, but the selection may look at the slot of the first
                    assert count == 0 and u + first < len(units) + nwg
                if least == so.t_min_range_groups(gu, slots):
                    assert count <= slots
                base += c


def test_static_rows():
    """About half of a unit's claims are static, whole ones, and never the last."""
    so = lib()
    C = so.t_claim_rows()
    for n in [0, 1, C - 1, C, C + 1, 2 * C - 1, 2 * C, 2 * C + 1, 7 * C, 16 * C + 5, 1 << 30]:
        s, claims = so.t_static_rows(n), -(-n // C)
        assert s % C == 0 and s == C * (claims // 2)
        assert s < n or n == 0


def test_added_min_range():
    """At most 32 groups, and at least 12 ranges for a unit of 12 groups or more."""
    so = lib()
    for gu in range(1, 3000):
        R = so.t_added_min_range(gu)
        assert 1 <= R <= 32
        assert R == 32 or -(-gu // R) <= 12
        assert R == 1 or gu > 12 * (R - 1)
