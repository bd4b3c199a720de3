"""The plan that cuts the keys of the rows beyond the last whole tile into parts: every key block in one part, a block per wave at least,
no more workgroups than units, sums within the scratch."""
import ctypes

import pytest
from test_staging_addresses import _load


def parts_of(n, hq, dh, cu, scratch):
    per = ctypes.c_int()
    return _load().dash_few_tail_parts(n, hq, dh, cu, ctypes.c_size_t(scratch), ctypes.byref(per)), per.value


def layer_scratch(n, K, N):
    """Bytes that the layer call has for the parts: the projection's scratch."""
    lib = _load()
    lib.dash_wo_scratch_bytes.restype = ctypes.c_size_t
    return lib.dash_wo_scratch_bytes(n, K, N)


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("hq", [1, 16, 28, 64, 300])
def test_every_block_once(hq, dh):
    for n in (1, 255, 256, 257, 300, 511, 513, 1025, 2305, 4097, 4351, 8200, 14001, 52429, 131071):
        rows, blocks = n % 256, -(-n // 32)
        for scratch in (0, 1 << 16, 1 << 20, 1 << 30):
            parts, per = parts_of(n, hq, dh, 256, scratch)
            assert parts >= 1 and -(-blocks // per) == parts
            if parts > 1:
                assert per % 8 == 0 and parts * -(-rows // 32) * hq <= 256
                assert parts * rows * hq * (dh + 2) * 4 <= scratch
    assert parts_of(4096, hq, dh, 256, 1 << 30)[0] == 1
