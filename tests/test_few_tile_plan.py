"""CPU check of the tiles for the fewest rows: their staging addresses, and the choice of rows per tile and K parts."""
import ctypes

import numpy as np
import pytest

from test_small_tile_plan import product_plan
from test_staging_addresses import _load


def few_plan(*args, **kw):
    p = product_plan(*args, **kw)
    return p.few_rows, p.tiles, p.parts, p.per


@pytest.mark.parametrize("bm", [16, 32, 48])
def test_loads_fetch_the_clamped_rows_and_columns(bm):
    lib = _load()
    lib.dash_check_few_tiles.argtypes = [ctypes.c_int] * 5 + [ctypes.POINTER(ctypes.c_longlong)]
    rng = np.random.default_rng(bm)
    shapes = [(1, 64, 8, 1), (15, 512, 64, 1), (16, 576, 72, 1), (17, 1088, 136, 2), (47, 448, 264, 1), (49, 2048, 64, 4), (177, 3584, 3584, 1), (33, 3584, 512, 4)]
    shapes += [(int(rng.integers(1, 300)), 64 * int(rng.integers(1, 40)), 8 * int(rng.integers(1, 60)), 1) for _ in range(15)]
    for M, K, N, parts in shapes:
        n = ctypes.c_longlong(0)
        assert lib.dash_check_few_tiles(M, K, N, bm, parts, ctypes.byref(n)) == 0, (M, K, N, bm, parts)
        assert n.value > 0


def test_the_choice():
    """One round of workgroups, every wave a step at least in K parts and eight at most, heads in one tile unless a second pass follows,
    sums and norms within the scratch; measured choices."""
    assert few_plan(177, 3584, 3584)[::2] == (48, 1) and few_plan(16, 3584, 3584)[::2] == (16, 4)
    assert few_plan(333, 512, 512)[::2] == (16, 1) and few_plan(333, 1024, 1024)[::2] == (32, 1)
    for M, K, N in ((64, 3584, 3584), (256, 3584, 3584), (1500, 512, 512), (2120, 3584, 3584), (16, 18944, 3584), (16, 3584, 37888)):
        assert few_plan(M, K, N)[0] == 0, (M, K, N)
    assert few_plan(177, 3584, 3584, scratch=0)[0] == 0 and few_plan(177, 3584, 3584, scratch=1)[0] == 0
    assert few_plan(177, 512, 1024, norms=0, head=64)[0] > 0 and few_plan(177, 512, 1024, norms=0, head=128)[0] == 0
    rng = np.random.default_rng(5)
    for _ in range(400):
        M, K, N = int(rng.integers(1, 1200)), 64 * int(rng.integers(1, 120)), 8 * int(rng.integers(1, 900))
        scratch, head = int(rng.integers(0, 3)) * (4 << 20), int(rng.choice([0, 64, 128]))
        bm, tiles, parts, per = few_plan(M, K, N, norms=1, head=head, scratch=scratch)
        if bm == 0:
            continue
        assert bm in (16, 32, 48) and tiles == -(-M // bm) * -(-N // 64) and tiles * parts <= 256 and M <= 1024
        assert (parts - 1) * per < K // 64 <= parts * per and per <= 64 and (parts == 1 or per >= 8)
        assert parts > 1 or head <= 64
        assert (parts * M * N * 4 if parts > 1 else -(-N // 64) * M * 8) <= scratch
