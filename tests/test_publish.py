"""CPU check of the words through which the workgroups of the one-launch score + decision + compaction kernel (rules NONE and THRESHOLD)
hand each other the chunks' decisions: a bounded wait that ended without its word fails the call. (TOPK's keys: test_topk_keys.py.)"""
import ctypes

import pytest

from test_staging_addresses import _load


def _step(chunks, splits, late, backwards=0):
    lib = _load()
    lib.dash_check_publish.argtypes = [ctypes.c_int] * 4 + [ctypes.POINTER(ctypes.c_int)]
    gathered = (ctypes.c_int * chunks)()
    return lib.dash_check_publish(chunks, splits, late, backwards, gathered), list(gathered)


@pytest.mark.parametrize("chunks", [1, 2, 3, 24, 70])
@pytest.mark.parametrize("backwards", [0, 1])
def test_a_late_publisher_fails_the_call(chunks, backwards):
    assert _step(chunks, 4, -1, backwards) == (sum(c % 65 for c in range(chunks)), [4] * chunks)
    for late in range(chunks):
        # chunks before it need none of its words, and its own publisher copies its own columns; nothing else is gathered. The count
        # is -1 also where a workgroup fails before or after the last chunk's, which may not have failed, writes it
        assert _step(chunks, 4, late, backwards) == (-1, [4] * late + [1] + [0] * (chunks - late - 1)), late
    assert _step(chunks, 1, chunks - 1, backwards) == (sum(c % 65 for c in range(chunks)), [1] * chunks)  # nobody waited for it
