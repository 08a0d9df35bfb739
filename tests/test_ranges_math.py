"""The scoring pass's ranges over valid groups, by brute force (no GPU).

Items (requests with ``mult`` units each) have vg groups per unit; groups are
numbered unit-major and cut into ranges of R = max(ceil(total / nwg),
min_range).  Every group must lie in exactly one of the nwg ranges, the
workgroups that meet a unit must be the ones between its first and last
group's, slot unit + workgroup must be unique and below U + nwg, and with the
least range length of a slot budget no unit may meet more ranges than it.
"""
from __future__ import annotations

import numpy as np
import pytest


def min_range(gu, max_slots):
    return (gu - 1) // (max_slots - 1) + 1


@pytest.mark.parametrize("items,mult,gu,nwg,slots", [
    (1, 1, 1, 1, 8), (16, 8, 188, 256, 8), (130, 1, 47, 256, 8), (70, 2, 300, 512, 8),
    (5, 3, 15, 64, 8), (16, 8, 1024, 512, 16), (3, 4, 2048, 256, 8), (9, 1, 8, 100, 2)])
def test_ranges(items, mult, gu, nwg, slots):
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
        total = int(units.sum())
        for least in (1, min_range(gu, slots)):
            R = max(-(-total // nwg), least)
            ranges = [(min(w * R, total), min((w + 1) * R, total)) for w in range(nwg)]
            assert sum(b - a for a, b in ranges) == total
            seen, base = set(), 0
            for u, g in enumerate(units):
                if g:
                    lo, hi = base // R, (base + int(g) - 1) // R
                    meets = [w for w, (a, b) in enumerate(ranges) if a < base + g and b > base]
                    assert meets == list(range(lo, hi + 1))
                    for w in meets:
                        assert u + w not in seen and u + w < len(units) + nwg
                        seen.add(u + w)
                    if least > 1:
                        assert hi - lo + 1 <= slots
                base += int(g)
