"""CPU check of the choice between attention's forms (one key group per workgroup, two, or the last rows apart)."""
import pytest

from test_staging_addresses import _load

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
