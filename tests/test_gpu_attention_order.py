"""Attention where its longest workgroups start in the second round: rows of every query tile and head against fp64."""
import numpy as np
import pytest
import torch

from paper_2604_18103_amd import binding as B
from test_attention_order import _later
from test_staging_addresses import _load

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,hq,hkv,dh", [(5121, 32, 8, 128), (6874, 28, 4, 128), (10000, 16, 8, 64), (12545, 12, 3, 128), (12001, 16, 16, 64)])
def test_rows_of_every_tile(n, hq, hkv, dh):
    """One row per 256 (its first, its last or one between) of every head: three bf16 roundings (scaled q, P, O), 2^-9 each
    of a row, so 2^-7 of the row's largest element covers them."""
    units, tiles = torch.cuda.get_device_properties(0).multi_processor_count, (n + 255) // 256
    assert _load().dash_fa_form(n, hq, dh, 1, units) != 1 and _later(n, hq, hkv, dh, units)[0] > 0
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


@pytest.mark.parametrize("n,hq,hkv", [(4900, 16, 4), (6595, 12, 4), (9999, 8, 8)])
def test_two_key_groups(n, hq, hkv):
    """128-row workgroups at head size 64: one row per workgroup of every head, held as the form's other cases are (three bf16
    roundings: 3.5e-3 of a row on the mean, 8e-3 on the largest)."""
    units = torch.cuda.get_device_properties(0).multi_processor_count
    assert _load().dash_fa_form(n, hq, 64, 1, units) == 1 and _later(n, hq, hkv, 64, units)[0] > 0
    g = torch.Generator(device="cuda").manual_seed(n)
    q, k, v = (torch.randn((n, h, 64), generator=g, device="cuda").bfloat16() for h in (hq, hkv, hkv))
    p = B.make_params(hq * 64, hq, hkv, 64, rule=B.RULE_NONE)
    o = torch.full((n, hq * 64), float("nan"), dtype=torch.bfloat16, device="cuda")
    B.dash_flash_fwd(p, q, k, v, torch.arange(n, dtype=torch.int32, device="cuda"), n, o)
    assert bool(torch.isfinite(o).all())
    tiles = (n + 127) // 128
    rows = np.minimum(np.arange(tiles) * 128 + np.random.default_rng(n).choice([0, 127, 77, 31], tiles), n - 1)
    rows = torch.from_numpy(np.unique(rows)).cuda()
    hidden = torch.arange(n, device="cuda")[None, :] > rows[:, None]
    err = []
    for h in range(hq):
        kh, vh = k[:, h // (hq // hkv)].double(), v[:, h // (hq // hkv)].double()
        s = (q[rows, h].double() @ kh.t().contiguous()) * 0.125
        want = torch.softmax(s.masked_fill_(hidden, float("-inf")), dim=1) @ vh
        err.append((o[rows][:, h * 64:(h + 1) * 64].double() - want).norm(dim=1) / want.norm(dim=1))
    err = torch.cat(err)
    assert float(err.max()) <= 8e-3 and float(err.mean()) <= 3.5e-3
