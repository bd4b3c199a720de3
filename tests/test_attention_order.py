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


def _later(n, hq, hkv, dh, units=256):
    """(how many start later, workgroups in one order, units of that order) of a causal launch over n rows in the form it takes."""
    groups = 2 if _load().dash_fa_form(n, hq, dh, 1, units) == 1 else 1
    slots = ctypes.c_int(0)
    later = _load().dash_fa_launch_later(-(-n * groups // 256), hq, hkv, dh, groups, units, ctypes.byref(slots))
    return later, slots.value, units // 8 if hkv in (1, 2, 4) or hkv % 8 == 0 else units


# measured figures: fa_deal_pays
@pytest.mark.parametrize("n,hq,hkv,dh,pays", [
    (20443, 8, 8, 128, 1), (10203, 16, 8, 128, 1), (13531, 16, 8, 128, 1), (5851, 28, 4, 128, 1), (6875, 28, 4, 128, 1), (5083, 32, 8, 128, 1),
    (6107, 32, 8, 128, 1), (14811, 12, 3, 128, 1), (3291, 48, 8, 128, 1), (12251, 16, 4, 64, 1), (7387, 24, 8, 64, 1), (4059, 40, 8, 64, 1),
    (4935, 16, 4, 64, 1), (6595, 12, 4, 64, 1), (10081, 8, 8, 64, 1),
    (2779, 64, 8, 64, 0), (3035, 64, 8, 128, 0), (2445, 32, 8, 64, 0), (5339, 40, 8, 128, 0), (9435, 24, 8, 64, 0), (9435, 16, 4, 64, 0), (13019, 12, 3, 64, 0),
    (4096, 28, 4, 128, 0), (8192, 28, 4, 128, 0), (16384, 28, 4, 128, 0)])
def test_where_it_pays(n, hq, hkv, dh, pays):
    assert (_later(n, hq, hkv, dh)[0] > 0) == bool(pays)


def test_a_launch_has_its_workgroups():
    """Those that wait are at most a round of units, and another round is behind them; an XCD's order covers its share of the items."""
    for hq, hkv in ((8, 8), (28, 4), (32, 8), (12, 3), (40, 8), (64, 16), (48, 6)):
        for dh in (64, 128):
            for n in range(300, 30000, 211):
                later, slots, units = _later(n, hq, hkv, dh)
                groups = 2 if _load().dash_fa_form(n, hq, dh, 1, 256) == 1 else 1
                items = -(-n * groups // 256) * hq
                assert 0 <= later <= units and (later == 0 or units + later <= slots)
                assert (slots == items) if units == 256 else (items <= 8 * slots < items + 8 * 8)
