"""CPU check of the 192 x 128 small tiles: staging addresses and tile map, and the rule that takes them."""
import ctypes

import numpy as np

from test_small_tile_plan import _lib, product_plan

TALL = 4


def tall_plan(M, K, N, cu=256, norms=1, scratch=1 << 26):
    p = product_plan(M, K, N, cu, norms, 0, scratch)
    return p.form, p.tiles


def test_staging_loads_fetch_the_clamped_rows_and_columns():
    lib, rng = _lib(), np.random.default_rng(4)
    shapes = [(1, 64, 8), (191, 128, 64), (192, 192, 72), (193, 64, 128), (383, 320, 136), (1220, 3584, 4608), (1700, 3584, 3584)]
    shapes += [(int(rng.integers(1, 900)), 64 * int(rng.integers(1, 12)), 8 * int(rng.integers(1, 90))) for _ in range(15)]
    for M, K, N in shapes:
        n = ctypes.c_longlong(0)
        assert lib.dash_check_small_staging(M, K, N, TALL, ctypes.byref(n)) == 0 and n.value > 0, (M, K, N)


def test_where_they_are_taken():
    """One round of workgroups, 16 K steps or more, and in place of two 128 x 128 workgroups per unit only."""
    for M, K, N in ((1153, 3584, 3584), (1728, 3584, 3584), (1220, 3584, 4608), (1536, 4096, 4096), (5000, 1024, 1024)):
        assert tall_plan(M, K, N)[0] == TALL, (M, K, N)
    assert tall_plan(1100, 3584, 3584)[0] == 2 and tall_plan(1800, 3584, 3584)[0] == 3
    assert tall_plan(1601, 960, 3584)[0] == 3 and tall_plan(16384, 3584, 3584)[0] == -1 and tall_plan(1400, 3584, 3584, scratch=0)[0] == -1
    rng = np.random.default_rng(5)
    for _ in range(300):
        M, K, N = int(rng.integers(1, 9000)), 64 * int(rng.integers(1, 80)), 8 * int(rng.integers(1, 800))
        form, tiles = tall_plan(M, K, N)
        assert form != TALL or (tiles == -(-M // 192) * -(-N // 128) <= 256 and K >= 1024)
