"""Attention where its longest workgroups start in the second round: rows of every query tile and head against fp64."""
import numpy as np
import pytest
import torch

from paper_2604_18103_amd import binding as B
from test_attention_order import _order

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,hq,hkv,dh", [(5121, 32, 8, 128), (6874, 28, 4, 128), (10000, 16, 8, 64), (12545, 12, 3, 64), (12001, 16, 16, 64)])
def test_rows_of_every_tile(n, hq, hkv, dh):
    """One row per 256 (its first, its last or one between) of every head: three bf16 roundings (scaled q, P, O), 2^-9 each
    of a row, so 2^-7 of the row's largest element covers them."""
    units, tiles = torch.cuda.get_device_properties(0).multi_processor_count, (n + 255) // 256
    slots, mine = (tiles * hq, units) if hkv == 3 else ((tiles * hq + 7) // 8, units // 8)
    assert _order(slots, mine) != list(range(slots))
    g = torch.Generator(device="cuda").manual_seed(n)
    q, k, v = (torch.randn((n, h, dh), generator=g, device="cuda").bfloat16() for h in (hq, hkv, hkv))
    idx = torch.arange(n, dtype=torch.int32, device="cuda")
    p = B.make_params(hq * dh, hq, hkv, dh, rule=B.RULE_NONE)
    o = torch.full((n, hq * dh), float("nan"), dtype=torch.bfloat16, device="cuda")
    B.dash_flash_fwd(p, q, k, v, idx, n, o)
    assert bool(torch.isfinite(o).all())
    rng = np.random.default_rng(n)
    rows = torch.from_numpy(np.unique(np.minimum(np.arange(tiles) * 256 + rng.choice([0, 255, 77, 130], tiles), n - 1))).cuda()
    hidden = torch.arange(n, device="cuda")[None, :] > rows[:, None]
    for h in range(hq):
        kh, vh = k[:, h // (hq // hkv)].double(), v[:, h // (hq // hkv)].double()
        s = (q[rows, h].double() @ kh.t().contiguous()) * dh ** -0.5
        want = torch.softmax(s.masked_fill_(hidden, float("-inf")), dim=1) @ vh
        got = o[rows][:, h * dh:(h + 1) * dh].double()
        assert bool(((got - want).abs() <= 2.0 ** -7 * want.abs().amax(dim=1, keepdim=True)).all()), h
