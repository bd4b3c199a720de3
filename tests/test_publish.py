"""CPU check of the words through which the one-launch score + decision + compaction kernel's workgroups hand each other the
chunks' decisions: a bounded wait that ended without its word fails the call."""
import ctypes

import pytest

from test_staging_addresses import _load


def _step(chunks, splits, late):
    lib = _load()
    lib.dash_check_publish.argtypes = [ctypes.c_int] * 3 + [ctypes.POINTER(ctypes.c_int)]
    gathered = (ctypes.c_int * chunks)()
    return lib.dash_check_publish(chunks, splits, late, gathered), list(gathered)


@pytest.mark.parametrize("chunks", [1, 2, 3, 24])
def test_a_late_publisher_fails_the_call(chunks):
    assert _step(chunks, 4, -1) == (sum(range(chunks)), [4] * chunks)
    for late in range(chunks if chunks > 1 else 0):  # the last one too: it finds every key itself
        # a first chunk whose publisher had every key copies its own columns; nothing else is gathered. The count is -1 also
        # where a workgroup fails before or after the last chunk's, which did not, would write it
        assert _step(chunks, 4, late) == (-1, [int(late == 0)] + [0] * (chunks - 1)), late
