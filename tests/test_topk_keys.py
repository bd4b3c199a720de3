"""CPU check of how a workgroup of the one-launch TopK kernel takes the keys of all rows: words that come late are asked for again, and
one that does not come is replaced by the key made from the row's norm pairs, so the call ends with every key whatever the order in which
workgroups get onto the chip."""
import ctypes

import pytest

from test_staging_addresses import _load


@pytest.mark.parametrize("n", [1, 63, 257, 1024, 1025, 2120, 4095, 4096])
def test_a_late_key_is_made_from_its_pairs(n):
    lib, own = _load(), ctypes.c_int()
    lib.dash_check_topk_keys.argtypes = [ctypes.c_int] * 4 + [ctypes.POINTER(ctypes.c_int)]
    asks = lib.dash_key_asks()
    for lo, hi in ((0, 0), (0, min(n, 64)), (n - n % 64, n), (0, n)):
        for late in (1, asks - 1, asks, -1):
            assert lib.dash_check_topk_keys(n, lo, hi, late, ctypes.byref(own)) == 0, (lo, hi, late)
            assert own.value == (hi - lo if late in (asks, -1) else 0), (lo, hi, late)
