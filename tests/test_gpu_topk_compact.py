"""The layer call's TOPK rule where workgroups exchange keys and each finds the cut itself: lengths at the edges of a chunk, of a
thread's keys (1024 rows each) and of the two forms (4096), with ties across those edges, against the oracle's TopK on the GPU's own
scores, bit for bit."""
import pytest

torch = pytest.importorskip("torch")
from test_gpu_topk_one_launch import _layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [514, 575, 577, 1023, 1025, 2047, 2049, 3072, 4095, 4096, 4097, 5121, 8191, 8192, 8193])
def test_against_the_oracle(n):
    for i, (k_keep, prot, kind) in enumerate(((n // 3, (0, 0), "spread"), (n, (0, 0), "spread"), (0, (0, 0), "spread"),
                                              (n - n // 5, (64, 32), "tied"), (n // 2 + 1, (1, 0), "few"), (3, (64, 32), "nan"))):
        _layer(n, 64, 1, k_keep, prot, kind, seed=n + i)


@pytest.mark.parametrize("n", [257, 300, 511, 512])
def test_wide_rows(n):
    """More than 32 norm pairs a row: an exchange from 257 rows on."""
    for k_keep, prot, kind in ((n // 3, (0, 0), "spread"), (n - 9, (64, 32), "tied")):
        _layer(n, 2120, 1, k_keep, prot, kind, seed=n)
