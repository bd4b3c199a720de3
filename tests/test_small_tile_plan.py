"""CPU check of the small-tile product: its staging addresses and tile map, and the choice of a form."""
import collections
import ctypes

import numpy as np
import pytest

from test_staging_addresses import _load

FORMS = range(4)


def _lib():
    lib = _load()
    lib.dash_check_small_staging.argtypes = [ctypes.c_int] * 4 + [ctypes.POINTER(ctypes.c_longlong)]
    lib.dash_check_small_staging.restype = ctypes.c_int
    lib.dash_product_plan.argtypes = [ctypes.c_int] * 6 + [ctypes.c_ulonglong, ctypes.POINTER(ctypes.c_int)]
    lib.dash_product_plan.restype = None
    return lib


Plan = collections.namedtuple("Plan", "form tiles parts per few_rows large_parts rest rest_parts")


def product_plan(M, K, N, cu=256, norms=1, head=0, scratch=1 << 26):
    """What the launcher decides about a product."""
    out = (ctypes.c_int * 8)()
    _lib().dash_product_plan(M, K, N, cu, norms, head, scratch, out)
    return Plan(*out)


def form_of(plan):
    """0 to 4: the small form; 16, 32, 48: rows of the few-row tiles; -1: large tiles."""
    return plan.few_rows or plan.form


@pytest.mark.parametrize("form", FORMS)
def test_staging_loads_fetch_the_clamped_rows_and_columns(form):
    lib = _lib()
    rng = np.random.default_rng(form)
    shapes = [(1, 64, 8), (63, 128, 64), (64, 192, 72), (65, 64, 128), (127, 320, 136), (129, 128, 264), (177, 3584, 3584),
              (333, 512, 512), (804, 3584, 4608), (64, 18944, 3584), (2120, 512, 1024)]
    shapes += [(int(rng.integers(1, 900)), 64 * int(rng.integers(1, 12)), 8 * int(rng.integers(1, 90))) for _ in range(15)]
    for M, K, N in shapes:
        n = ctypes.c_longlong(0)
        assert lib.dash_check_small_staging(M, K, N, form, ctypes.byref(n)) == 0, (M, K, N, form)
        assert n.value > 0


def test_left_over_tiles_in_k_parts():
    """Half tiles left over after the whole rounds are cut along K when there are few of them and scratch holds the sums."""
    lib = _load()
    lib.dash_rest_parts.argtypes = [ctypes.c_int] * 4 + [ctypes.c_ulonglong]
    parts = lambda *a: lib.dash_rest_parts(*a)
    assert parts(4700, 3584, 3584, 256, 1 << 26) > 2 and parts(4700, 18944, 3584, 256, 1 << 26) > 4
    assert parts(16384, 3584, 3584, 256, 1 << 26) == 1          # 128 left over fill the units as they are
    assert parts(4700, 3584, 3584, 256, 0) == 1                 # no scratch
    assert parts(4700, 3584, 3584, 256, 3 * 20 * 131072) <= 3   # as many as the scratch holds
    assert parts(4700, 512, 3584, 256, 1 << 26) == 1            # too few steps to cut
    for M, K, N in ((4700, 3584, 3584), (4700, 18944, 3584), (9500, 3584, 3584), (400, 3584, 37888), (3700, 3584, 4608)):
        n = ctypes.c_longlong(0)
        assert parts(M, K, N, 256, 1 << 26) > 1
        assert lib.dash_check_gemm_staging(M, K, N, 256, 1 << 26, ctypes.byref(n)) == 0


def test_choice_of_a_form():
    """Large products keep the large tiles; short ones take small tiles or the few-row ones, along K in parts only where the tiles
    alone leave the chip idle; without scratch none."""
    def plan(M, K, N, norms=1, scratch=1 << 30):
        p = product_plan(M, K, N, norms=norms, scratch=scratch)
        return (form_of(p), *p[1:4])

    for M, K, N in ((16384, 3584, 3584), (8192, 3584, 4608), (4097, 3584, 3584), (32768, 3584, 37888), (8192, 18944, 3584)):
        assert plan(M, K, N)[0] == -1, (M, K, N)
    assert plan(177, 3584, 3584)[0] >= 0 and plan(177, 3584, 3584)[2] == 1
    assert plan(333, 512, 512)[0] >= 0 and plan(333, 512, 512)[2] == 1
    assert plan(64, 18944, 3584)[2] > 1                       # a long contraction of few tiles: parts
    assert plan(177, 3584, 3584, scratch=0)[0] == -1          # row norms need scratch
    assert plan(177, 3584, 4608, norms=0, scratch=0)[0] == -1  # one order of the K steps
    assert plan(177, 3584, 4608, norms=0, scratch=1)[2] == 1   # room for nothing: no parts
    assert plan(177, 3584, 3584, norms=1, scratch=1)[0] == -1  # nor for row norms
    rng = np.random.default_rng(7)
    for _ in range(300):
        M, K, N = int(rng.integers(1, 6000)), 64 * int(rng.integers(1, 300)), 8 * int(rng.integers(1, 5000))
        scratch = int(rng.integers(0, 3)) * (8 << 20)
        form, tiles, parts, per = plan(M, K, N, int(rng.integers(0, 2)), scratch)
        if form >= 0:
            assert parts >= 1 and (parts - 1) * per < K // 64 <= parts * per
            assert parts == 1 or parts * M * N * 4 <= scratch


def test_no_xcd_gets_more_than_an_eighth():
    """A launch in K parts is planned to fit the units in one round; with workgroup b on XCD b % 8, that holds only if no
    XCD gets more workgroups than it has units."""
    lib = _lib()
    lib.dash_small_deal.argtypes = [ctypes.c_int] * 2
    lib.dash_small_deal.restype = ctypes.c_int
    for tiles in range(1, 257):
        for parts in range(1, 256 // tiles + 1):
            assert lib.dash_small_deal(tiles, parts) == (tiles * parts + 7) // 8, (tiles, parts)
    for tiles in (300, 476, 512, 1000, 2047):
        assert lib.dash_small_deal(tiles, 1) == (tiles + 7) // 8


def test_small_tiles_only_for_products_of_few_large_tiles():
    """Products of more than two large row tiles whose large tiles occupy more than half of the units keep them: several
    rounds of small tiles were up to 1.3 times as slow."""
    rng = np.random.default_rng(11)
    shapes = [(513, 3584, 18944), (4700, 320, 3584), (8001, 320, 2112), (6600, 3584, 2080), (12001, 512, 6144)]
    shapes += [(int(rng.integers(1, 20000)), 64 * int(rng.integers(1, 300)), 8 * int(rng.integers(1, 5000))) for _ in range(400)]
    for M, K, N in shapes:
        p = product_plan(M, K, N, scratch=1 << 30)
        if M > 512 and 2 * (-(-M // 256)) * (-(-N // 256)) > 256:
            assert p.form == -1 and p.few_rows in (0, 16, 32, 48) and (p.few_rows == 0 or M <= 1024), (M, K, N, p)
    assert product_plan(17, 3584, 37888, norms=0, scratch=1 << 30).form >= 0
