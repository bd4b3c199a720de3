"""CPU check of the choice between attention's forms (one key group per workgroup, two, or the last rows apart), and of what the
form with two key groups fetches and when."""
import ctypes
import os
import subprocess

import pytest

from test_staging_addresses import PKG, _load

ONE, TWO, ONE_AND_TAIL = 0, 1, 2


# measured without a causal mask, 256 compute units, the other form / this one: 8001 823 / 758 us, 5500 406 / 384, 32 heads
# 6600 675 / 647; 2400 111 / 101, 14001 0.967 times; 16 heads of 64: 4300 137 / 122, 4097 112 / 107
@pytest.mark.parametrize("n,hq,dh,causal,form", [
    (5500, 28, 128, 0, ONE), (7424, 28, 128, 0, ONE), (7500, 28, 128, 0, ONE), (8001, 28, 128, 0, ONE),
    (4352, 32, 128, 0, ONE), (4700, 32, 128, 0, ONE), (6600, 32, 128, 0, ONE), (7000, 32, 128, 0, ONE),
    (2400, 28, 128, 0, ONE_AND_TAIL), (14001, 28, 128, 0, ONE_AND_TAIL), (4100, 32, 128, 0, ONE_AND_TAIL),
    (4097, 16, 64, 0, ONE_AND_TAIL), (1152, 28, 128, 0, TWO), (4480, 16, 64, 0, TWO), (9700, 16, 64, 0, TWO), (14001, 16, 64, 0, ONE), (1500, 28, 128, 0, ONE),
    (2304, 28, 128, 1, TWO), (2400, 28, 128, 1, ONE), (4096, 16, 64, 1, TWO), (16384, 28, 128, 1, ONE)])
def test_the_faster_form(n, hq, dh, causal, form):
    assert _load().dash_fa_form(n, hq, dh, causal, 256) == form


def test_nearly_equal_counts_keep_one_group():
    """0.57 times the rounds of 128-row workgroups within 6 % of the rounds of 256-row ones: one key group."""
    lib = _load()
    for n in range(1, 20000, 7):
        for hq in (4, 16, 28, 32):
            one, two = -(-(-(-n // 256) * hq) // 256), -(-(-(-n // 128) * hq) // 256)
            if 0.57 * two > 0.945 * one:
                assert lib.dash_fa_form(n, hq, 128, 0, 256) != TWO, (n, hq)


def _groups(lib, n, hkv, dh, causal, row0, row1):
    lib.dash_check_flash_groups.argtypes = [ctypes.c_int] * 6 + [ctypes.POINTER(ctypes.c_longlong)]
    loads = ctypes.c_longlong(0)
    return lib.dash_check_flash_groups(n, hkv, dh, causal, row0, row1, ctypes.byref(loads)), loads.value


@pytest.mark.parametrize("n", [1, 63, 64, 65, 127, 128, 129, 192, 193, 255, 256, 257, 300, 333, 513, 1000, 2120, 4097, 4224, 5000])
def test_two_key_groups_fetch_every_tile_once_and_in_time(n):
    lib = _load()
    for hkv, dh in ((4, 128), (1, 64), (2, 128)):
        for causal in (1, 0):
            status, loads = _groups(lib, n, hkv, dh, causal, 0, n)
            assert status == 0 and loads > 0, (n, hkv, dh, causal, status)
        if n > 256 and n % 256:  # the rows beyond the last whole tile as a launch of their own
            assert _groups(lib, n, hkv, dh, 0, n - n % 256, n)[0] == 0


@pytest.mark.parametrize("good,bad,n", [
    ("fa_k_lead(int grp) { return grp == 0 ? 1 : 2; }", "fa_k_lead(int grp) { return grp == 0 ? 1 : 3; }", 1000),
    ("fa_v_lead(int grp) { return grp == 0 ? 0 : 1; }", "fa_v_lead(int grp) { return grp == 0 ? 1 : 1; }", 1000),
    ("(all_tiles - grp + 1) / 2; }", "(all_tiles + 1) / 2; }", 64),
    ("2 * t + grp) * kFaBN; }", "2 * t) * kFaBN; }", 300)])
def test_a_planted_mistake_shows(good, bad, n, tmp_path):
    """A request a round too early, a tile count without the group, a group on the other's tiles: in a copy of the header."""
    src = open(os.path.join(PKG, "csrc", "staging_addr.h")).read()
    assert src.count(good) == 1
    (tmp_path / "staging_addr.h").write_text(src.replace(good, bad))
    (tmp_path / "staging_check.cpp").write_text(open(os.path.join(PKG, "csrc", "staging_check.cpp")).read())
    out = str(tmp_path / "libbad.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", str(tmp_path / "staging_check.cpp"), "-o", out], check=True)
    assert _groups(_load(out), n, 2, 64, 1, 0, n)[0] != 0
