"""CPU check of attention's few-row form: where it is taken, and that its waves fetch every key block once and in range."""
import ctypes
import os
import subprocess

import pytest

from test_staging_addresses import PKG, _load


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


def _queries(lib, n, hq, dh, waves, row_base):
    loads = ctypes.c_longlong(0)
    lib.dash_check_few_queries.argtypes = [ctypes.c_int] * 5 + [ctypes.POINTER(ctypes.c_longlong)]
    return lib.dash_check_few_queries(n, hq, dh, waves, row_base, ctypes.byref(loads)), loads.value


@pytest.mark.parametrize("n,row_base", [(1, 0), (31, 0), (32, 0), (33, 0), (64, 0), (95, 0), (333, 0), (2305, 2304), (2335, 2304), (2336, 2304),
                                        (2337, 2304), (4097, 4096), (2559, 2304), (4351, 4096)])
def test_query_rows_once_and_in_range(n, row_base):
    """Launches over all rows, and over those beyond the last whole 256-row tile."""
    for hq, dh in ((28, 128), (3, 64), (1, 128)):
        for waves in (4, 8):
            status, loads = _queries(_load(), n, hq, dh, waves, row_base)
            assert status == 0 and loads == -(-(n - row_base) // 32) * hq * 32 * dh // 8, (n, hq, dh, waves, status)


@pytest.mark.parametrize("good,bad", [
    ("r, sa_min(n - row0, kFewKeys), Hq, DH);", "r, kFewKeys, Hq, DH);"),                       # no clamp at the last row
    ("return wave * few_q_loads(DH, KW) + u; }", "return wave + u; }"),                         # two waves on one piece
    ("(size_t)(row0 / kFewKeys) * few_block_bytes(Hq, DH); }", "(size_t)(row0 % 256 / kFewKeys) * few_block_bytes(Hq, DH); }")])  # the tail's base
def test_a_planted_mistake_shows(good, bad, tmp_path):
    src = open(os.path.join(PKG, "csrc", "staging_addr.h")).read()
    assert src.count(good) == 1
    (tmp_path / "staging_addr.h").write_text(src.replace(good, bad))
    (tmp_path / "staging_check.cpp").write_text(open(os.path.join(PKG, "csrc", "staging_check.cpp")).read())
    out = str(tmp_path / "libbad.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", str(tmp_path / "staging_check.cpp"), "-o", out], check=True)
    assert any(_queries(_load(out), 2305, 2, 128, 4, base)[0] != 0 for base in (0, 2304))


# this form / the tiled kernels, us, 256 units: the figures at few_waves
@pytest.mark.parametrize("n,hq,dh,causal,waves", [
    (17, 28, 128, 1, 8), (192, 28, 128, 1, 8), (320, 28, 128, 1, 4), (832, 28, 128, 1, 4), (960, 28, 128, 1, 0),
    (3072, 8, 128, 1, 4), (4096, 8, 128, 1, 0), (1024, 16, 64, 1, 8), (2560, 16, 64, 1, 4), (2816, 16, 64, 1, 0),
    (576, 28, 128, 0, 4), (640, 28, 128, 0, 0), (1024, 16, 64, 0, 8), (1152, 16, 64, 0, 0), (16384, 28, 128, 1, 0)])
def test_the_faster_form(n, hq, dh, causal, waves):
    assert _load().dash_few_waves(n, hq, dh, causal, 256) == waves
