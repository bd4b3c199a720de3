"""q/k/v projections with the rotary embedding in the product's epilogue, through every form the product takes."""
import numpy as np
import pytest
import torch

from paper_2604_18103_amd import binding as B
from test_small_tile_plan import form_of, product_plan

pytestmark = pytest.mark.gpu


def _rand(rng, shape, scale=1.0):
    return torch.from_numpy((rng.standard_normal(shape) * scale).astype(np.float32)).bfloat16().cuda()


def _rotate(u, pos, theta):
    half = u.shape[2] // 2
    a = pos.double()[:, None] * theta ** (-torch.arange(half, device=u.device, dtype=torch.float64) / half)
    c, s = torch.cos(a)[:, None], torch.sin(a)[:, None]
    lo, hi = u[..., :half], u[..., half:]
    return torch.cat([lo * c - hi * s, lo * s + hi * c], dim=2)


# rows, width, query / key-value heads, head size: few-row, 64x64, 64x128 and 128x128 tiles (one and two workgroups per unit), K parts,
# whole tiles, half tiles, left-over tiles in K parts
SHAPES = [(1, 64, 1, 1, 64), (65, 512, 6, 1, 64), (129, 512, 4, 2, 128), (70, 3584, 4, 2, 128), (70, 3584, 6, 1, 64),
          (333, 1024, 28, 4, 128), (804, 1024, 28, 4, 128), (1300, 512, 28, 4, 128), (2500, 3584, 28, 4, 128),
          (3612, 3584, 28, 4, 128), (4700, 512, 24, 8, 64), (5100, 512, 28, 4, 128)]


# the form each of these takes with the scratch left after the table: small form (0 to 4) or rows of the few-row tiles (16, 32, 48) and its
# K parts; -1 (large tiles), their K parts, whether half tiles are left over, and those in K parts
PLANNED = [((65, 512, 6, 1, 64), (16, 1)), ((300, 1024, 28, 4, 64), (48, 1)), ((70, 3584, 6, 1, 64), (32, 7)),
           ((70, 3584, 4, 2, 128), (48, 7)), ((16, 8192, 28, 4, 128), (16, 3)), ((1628, 832, 7, 1, 64), (0, 1)),
           ((1089, 320, 1, 1, 64), (0, 1)), ((733, 832, 16, 2, 64), (0, 1)), ((252, 7360, 5, 1, 64), (0, 9)),
           ((103, 5248, 16, 4, 64), (0, 5)), ((312, 3264, 4, 1, 128), (0, 4)), ((53, 2880, 32, 4, 128), (0, 3)),
           ((600, 1024, 28, 4, 64), (1, 1)), ((333, 1024, 28, 4, 128), (1, 1)), ((208, 6080, 16, 4, 64), (1, 5)),
           ((289, 2432, 16, 4, 128), (1, 2)), ((804, 1024, 56, 8, 64), (2, 1)), ((804, 1024, 28, 4, 128), (2, 1)),
           ((2000, 512, 28, 4, 64), (3, 1)), ((1300, 512, 28, 4, 128), (3, 1)), ((1400, 2048, 28, 4, 128), (3, 1)),
           ((1345, 1088, 52, 2, 64), (4, 1)), ((1200, 1024, 28, 4, 128), (4, 1)), ((300, 14336, 56, 8, 64), (-1, 7, False, 1)),
           ((300, 14336, 28, 4, 128), (-1, 7, False, 1)), ((2500, 3584, 56, 8, 64), (-1, 1, False, 1)),
           ((3612, 1024, 56, 8, 64), (-1, 1, True, 1)), ((5100, 512, 28, 4, 128), (-1, 1, True, 1)),
           ((3612, 3584, 56, 8, 64), (-1, 1, True, 6)), ((3612, 3584, 28, 4, 128), (-1, 1, True, 6))]


@pytest.mark.parametrize("shape,form", PLANNED)
def test_every_form_against_fp64(shape, form):
    """Both head sizes in every form of the product: the partner column lies 32 or 64 columns away, in the same tile, the
    neighbouring wave's, or another lane's of the second pass."""
    n, d, hq, hkv, dh = shape
    p = B.make_params(d, hq, hkv, dh, rule=B.RULE_NONE)
    scratch = B.qkv_workspace_bytes(p, n) - (n * (dh // 2) * 8 + 255) // 256 * 256
    units = torch.cuda.get_device_properties(0).multi_processor_count
    plan = product_plan(n, d, (hq + 2 * hkv) * dh, units, 0, dh, max(scratch, 1))
    got = (form_of(plan), plan.parts) if form_of(plan) >= 0 else (-1, plan.large_parts, plan.rest > 0, plan.rest_parts)
    assert got == form
    test_against_fp64(n, d, hq, hkv, dh)


@pytest.mark.parametrize("n,d,hq,hkv,dh", SHAPES)
def test_against_fp64(n, d, hq, hkv, dh):
    """One bf16 rounding of the rotated fp32 sums (2-norm of a row below 2^-8; measured 1.7e-3), h rounded to bf16 on the way
    as the library does it; and the two separate calls, which round q and k twice, within two roundings."""
    rng, theta = np.random.default_rng(n), 1.0e6
    p = B.make_params(d, hq, hkv, dh, rule=B.RULE_NONE)
    x, w = _rand(rng, (n, d), 2.0), _rand(rng, (d, (hq + 2 * hkv) * dh), d ** -0.5)
    pos = torch.from_numpy(np.sort(rng.permutation(131072)[:n]).astype(np.int32)).cuda()
    ws = torch.empty((max(B.qkv_workspace_bytes(p, n), 256),), dtype=torch.uint8, device="cuda")
    new = lambda: tuple(torch.zeros((n, h, dh), dtype=torch.bfloat16, device="cuda") for h in (hq, hkv, hkv))
    one, two, bare = new(), new(), new()
    h = torch.empty_like(x)
    B.dash_rmsnorm_qkv_rope(p, x, w, pos, n, theta, *one, h, ws)
    B.dash_rmsnorm_qkv_fused(p, x, w, n, *two, torch.empty_like(x), ws)
    B.dash_rope_qk(p, two[0], two[1], pos, n, theta)
    B.dash_rmsnorm_qkv_rope(p, x, w, pos, n, theta, *bare, torch.empty_like(x), None)   # no scratch: the two calls
    hd = h.double()
    assert float((hd - x.double() * torch.rsqrt(x.double().pow(2).mean(dim=1, keepdim=True) + 1e-6)).norm() / hd.norm()) <= 2.0 ** -8
    for i, wt in enumerate(w.split([hq * dh, hkv * dh, hkv * dh], dim=1)):
        want = (hd @ wt.double()).reshape(n, -1, dh)
        if i < 2:
            want = _rotate(want, pos, theta)
        for got, tol in ((one[i], 2.0 ** -8), (two[i], 2.0 ** -7), (bare[i], 2.0 ** -7)):
            err = (got.double() - want).reshape(n, -1).norm(dim=1) / want.reshape(n, -1).norm(dim=1)
            assert float(err.max()) <= tol, (i, float(err.max()))
    # the rotation keeps the length of every pair; v is not rotated
    assert torch.equal(one[2], two[2]) or float((one[2].double() - two[2].double()).norm() / two[2].double().norm()) <= 2.0 ** -8


def test_refused_calls():
    p = B.make_params(128, 2, 1, 64, rule=B.RULE_NONE)
    t = torch.zeros((4, 128), dtype=torch.bfloat16, device="cuda")
    w = torch.zeros((128, 256), dtype=torch.bfloat16, device="cuda")
    idx = torch.arange(4, dtype=torch.int32, device="cuda")
    for args in ((idx, 4, 0.5), (idx, -1, 1e6), (None, 4, 1e6)):
        with pytest.raises(B.DashError):
            B.dash_rmsnorm_qkv_rope(p, t, w, *args, t, t, t, t, None)
