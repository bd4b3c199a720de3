"""CPU check of the order in which attention's workgroups start: every item once, and by list scheduling no later an end than
heaviest first."""
import ctypes
import heapq

import pytest

from test_staging_addresses import _load


def _order(slots, units):
    out = (ctypes.c_int * slots)()
    _load().dash_fa_order(slots, units, out)
    return list(out)


def _end(lengths, units, cost):
    ends = [0.0] * units
    for t in lengths:
        heapq.heappush(ends, heapq.heappop(ends) + t + cost)
    return max(ends)


@pytest.mark.parametrize("units", [1, 2, 8, 32, 38, 256, 304])
def test_every_item_once(units):
    for slots in [s for s in range(1, 4 * units + 3) if units < 100 or s % 7 == 0]:
        assert sorted(_order(slots, units)) == list(range(slots))


@pytest.mark.parametrize("heads,step", [(1, 1), (2, 1), (4, 1), (7, 2), (16, 2)])
def test_no_later_than_heaviest_first(heads, step):
    """`heads` query heads on `step` XCDs of 32 units, one workgroup per head and query tile."""
    gain = 0.0
    for tiles in range(8, 150):
        heaviest = [t for t in range(tiles, 0, -1) for _ in range(heads)]
        slots = (len(heaviest) + step - 1) // step
        order = _order(slots, 32)
        for cost in (0.5, 0.8):
            for xcd in range(step):
                mine = [heaviest[i * step + xcd] for i in order if i * step + xcd < len(heaviest)]
                first, now = _end(heaviest[xcd::step], 32, cost), _end(mine, 32, cost)
                assert now <= first + 1e-9 + (1.0 if order == sorted(order) else 0.0), (tiles, cost)
                gain = max(gain, 1.0 - now / first)
    assert gain > 0.02
