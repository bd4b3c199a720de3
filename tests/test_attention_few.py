"""CPU check of attention's few-row form: where it is taken, and that its waves fetch every key block once and in range."""
import ctypes

import pytest

from test_staging_addresses import _load


def _check(n, hkv, dh, causal, waves):
    lib, loads = _load(), ctypes.c_longlong(0)
    lib.dash_check_flash_few.argtypes = [ctypes.c_int] * 5 + [ctypes.POINTER(ctypes.c_longlong)]
    return lib.dash_check_flash_few(n, hkv, dh, causal, waves, ctypes.byref(loads)), loads.value


@pytest.mark.parametrize("n", [1, 31, 32, 33, 64, 65, 127, 129, 255, 257, 333, 1025])
def test_every_block_once_and_in_range(n):
    for hkv, dh in ((4, 128), (1, 64), (2, 128)):
        for causal in (1, 0):
            if n > 500 and hkv > 1:
                continue
            for waves in (4, 8):
                status, loads = _check(n, hkv, dh, causal, waves)
                assert status == 0 and loads > 0, (n, hkv, dh, causal, waves, status)


# this form / the tiled kernels, us, 256 units: the figures at few_waves
@pytest.mark.parametrize("n,hq,dh,causal,waves", [
    (17, 28, 128, 1, 8), (192, 28, 128, 1, 8), (320, 28, 128, 1, 4), (832, 28, 128, 1, 4), (960, 28, 128, 1, 0),
    (3072, 8, 128, 1, 4), (4096, 8, 128, 1, 0), (1024, 16, 64, 1, 8), (2560, 16, 64, 1, 4), (2816, 16, 64, 1, 0),
    (576, 28, 128, 0, 4), (640, 28, 128, 0, 0), (1024, 16, 64, 0, 8), (1152, 16, 64, 0, 0), (16384, 28, 128, 1, 0)])
def test_the_faster_form(n, hq, dh, causal, waves):
    assert _load().dash_few_waves(n, hq, dh, causal, 256) == waves
