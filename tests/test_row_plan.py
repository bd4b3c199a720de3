"""CPU check of the lower tiles that a product's last round may take: where, that the launches cover every row once and stay in range."""
import ctypes

import pytest

from test_staging_addresses import _load


def _plan(M, K, N):
    out = (ctypes.c_int * 2)()
    lib = _load()
    lib.dash_row_plan.argtypes = [ctypes.c_int] * 4 + [ctypes.c_ulonglong, ctypes.POINTER(ctypes.c_int)]
    lib.dash_row_plan(M, K, N, 256, 64 << 20, out)
    return tuple(out)


# measured figures: row_plan
@pytest.mark.parametrize("M,K,N,rb,whole", [
    (2400, 3584, 3584, 6, 0), (3456, 3584, 3584, 6, 0), (3457, 3584, 3584, 7, 0), (4032, 3584, 3584, 7, 0), (4033, 3584, 3584, 0, 0),
    (2305, 3584, 4608, 6, 0), (2688, 3584, 4608, 6, 0), (7500, 18944, 3584, 6, 18), (8192, 18944, 3584, 7, 18), (11885, 18944, 3584, 6, 36),
    (11885, 3584, 3584, 0, 0), (8192, 3584, 3584, 0, 0), (9216, 18944, 3584, 0, 0), (16384, 3584, 3584, 0, 0), (8192, 1024, 1536, 0, 0), (1742, 2048, 8192, 7, 0), (3539, 4096, 4096, 7, 0), (7630, 14336, 4096, 0, 0), (11731, 14336, 4096, 0, 0), (7000, 14336, 4096, 6, 16), (6874, 18944, 3584, 0, 0)])
def test_where(M, K, N, rb, whole):
    assert _plan(M, K, N) == (rb, whole)


def test_every_row_once_and_in_range():
    lib = _load()
    taken = 0
    for K, N in ((3584, 3584), (18944, 3584), (512, 7168), (4096, 4096), (14336, 4096), (3584, 4608), (8192, 2056)):
        for M in list(range(1800, 14000, 131)) + [2305, 3456, 3457, 4032, 8192, 11885]:
            rb, whole = _plan(M, K, N)
            if rb == 0:
                continue
            taken += 1
            assert rb in (6, 7) and whole * 256 < M
            assert -(-(M - 256 * whole) // (32 * rb)) * -(-N // 256) <= 256
            if whole:
                assert lib.dash_check_rows(M, K, N, 0, whole * 256, 8) == 0, (M, K, N)
            assert lib.dash_check_rows(M, K, N, whole * 256, M, rb) == 0, (M, K, N)
    assert taken > 100


@pytest.mark.parametrize("M,K,N,rb", [(1486, 8192, 8192, 6), (1486, 256, 8192, 6), (1486, 4096, 6144, 6), (2400, 3584, 3584, 6)])
def test_an_xcd_reads_few_columns(M, K, N, rb):
    """Up to 8 row tiles, and where they are no multiple of 8: 32 consecutive tiles of panels of four columns and at least seven rows,
    which are parts of at most three panels."""
    assert _plan(M, K, N) == (rb, 0) and -(-M // (32 * rb)) >= 7
    assert _load().dash_rows_columns(N, 0, M, rb) <= 12


@pytest.mark.parametrize("M,K,N", [(3027, 2048, 4096), (6099, 512, 1536), (4563, 1024, 2048)])
def test_an_xcd_reads_whole_rows(M, K, N):
    """16 row tiles and more in eights: the plain order, every column of an eighth of the rows."""
    assert _plan(M, K, N) == (6, 0) and _load().dash_rows_columns(N, 0, M, 6) == N // 256
