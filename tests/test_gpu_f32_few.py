"""The fp32 projection on either side of the line between its 16-row and 32-row tiles, and contractions that end inside the chunks a
wave has in flight."""
import pytest
import torch

from test_gpu_f32 import test_f32_projection_tile_edges as _projection

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,hq,dh,d", [(1, 1, 64, 16452), (31, 4, 64, 8260), (33, 1, 128, 5508), (70, 2, 128, 3332)])
def test_32_row_tiles(n, hq, dh, d):
    """One 16-row tile too many for the units."""
    assert -(-n // 16) * -(-d // 64) > torch.cuda.get_device_properties(0).multi_processor_count
    _projection(n, hq, dh, d)


@pytest.mark.parametrize("n,hq,dh,d", [(5, 7, 64, 132), (16, 8, 64, 64), (17, 9, 64, 260), (47, 9, 128, 68), (130, 17, 64, 1024), (64, 2, 64, 4096)])
def test_16_row_tiles(n, hq, dh, d):
    """28, 32, 36, 72 and 68 chunks over 8 waves with four in flight; the last with exactly as many tiles as units. The bound of that
    test is for K <= 256 terms; the error of a sum grows no faster than their number, and eight waves share it: K / 8 <= 256."""
    assert -(-n // 16) * -(-d // 64) <= torch.cuda.get_device_properties(0).multi_processor_count
    _projection(n, hq, dh, d)
