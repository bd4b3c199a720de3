"""The layer call's TOPK rule where every workgroup decides about all rows itself: lengths at the edges of its chunks and of its
range, cuts inside groups of equal scores, against the oracle's TopK on the GPU's own scores, bit for bit."""
import pytest

from test_gpu_topk_one_launch import _layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["spread", "tied", "nan", "few"])
@pytest.mark.parametrize("n", [2, 65, 128, 192, 255, 256, 257, 320, 448, 511, 512, 513])
def test_every_cut(n, kind):
    """Nothing kept, one, all but one, all; a cut inside the second half of a chunk; the protected rows alone, and more of them
    than there are rows."""
    for i, (k_keep, prot) in enumerate(((0, (0, 0)), (1, (0, 0)), (n - 1, (0, 0)), (n, (0, 0)), (n // 2 + 5, (0, 0)),
                                        (min(n, 7), (min(n, 5), min(n, 2))), (min(n, 3), (n, 3)), ((2 * n) // 3, (1, 64)))):
        _layer(n, 128 if n % 2 else 1032, 1, min(k_keep, n), prot, kind, seed=n + i)


@pytest.mark.parametrize("n,d,hq", [(256, 8192, 1), (257, 8192, 1), (512, 8192, 2), (512, 4096, 2), (257, 4104, 2), (400, 8192, 128), (257, 16384, 1),
                                    (257, 2048, 1), (512, 2048, 1), (257, 2056, 1), (512, 2056, 1)])
def test_wide_rows(n, d, hq):
    """Up to 256 rows, and with 32 pairs of a row, 33 and more beyond that: keys that are handed over, or not; with 128 heads the product's
    large tiles leave fewer pairs than the width has columns of 64."""
    for i, (k_keep, prot, kind) in enumerate(((n // 3, (0, 0), "spread"), (n - 1, (5, 7), "spread"), (n // 2 + 5, (0, 0), "few"))):
        _layer(n, d, hq, k_keep, prot, kind, seed=n + i)
