"""The small-tile product in each of its forms, at the edges of the tiles and of the K groups, with every epilogue, against
fp64 sums of the same bf16 operands. The forms are what the launcher itself decides (product_plan)."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2604_18103_amd import binding as B
from test_small_tile_plan import _lib, form_of, product_plan

pytestmark = pytest.mark.gpu

# (rows, query heads of 64, width, the form (0 to 4: 64x64, 64x128, 128x128 with one and with two workgroups per unit, 192x128; 16: few-row
# tiles of 16 rows), K parts)
PROJECTIONS = [(1, 1, 64, 16, 1), (65, 3, 200, 16, 1), (129, 8, 512, 16, 1), (16, 300, 520, 16, 19),
               (149, 1, 3328, 0, 1), (1089, 5, 72, 0, 1), (2111, 9, 200, 0, 1), (293, 24, 3072, 0, 1), (632, 108, 1600, 0, 1),
               (305, 50, 896, 0, 3), (359, 57, 544, 0, 4),
               (333, 56, 3584, 1, 1), (1300, 16, 1000, 1, 1), (70, 56, 3584, 1, 4), (804, 56, 3584, 2, 1), (2200, 8, 1032, 2, 1),
               (5003, 9, 1096, 3, 1), (1873, 46, 3216, 3, 1), (2459, 38, 2968, 3, 1), (1601, 56, 3584, 4, 1)]


def _plan(M, K, N, norms, scratch, head=0):
    p = product_plan(M, K, N, torch.cuda.get_device_properties(0).multi_processor_count, norms, head, scratch)
    return (form_of(p), *p[1:4])


def _rand(rng, shape, scale=1.0):
    return torch.from_numpy((rng.standard_normal(shape) * scale).astype(np.float32)).bfloat16().cuda()


@pytest.mark.parametrize("n,heads,d,form,parts", PROJECTIONS)
def test_projection(n, heads, d, form, parts):
    """x_next: one bf16 rounding (2^-9 of the element; the bound is 2^-8 for a sum on the other side of a tie) beside fp32
    sums of K products (1e-5 of the largest); norms: fp32 sums of d squares, 1e-4 covers K and d terms in any order. The
    same call without scratch takes the large tiles: the same sums but for their order."""
    K, rng = heads * 64, np.random.default_rng(n + d)
    a, w, x = _rand(rng, (n, K)), _rand(rng, (K, d), K ** -0.5), _rand(rng, (n, d), 3.0)
    p = B.make_params(d, heads, 1, 64, rule=B.RULE_NONE)
    ws = torch.empty((64 << 20,), dtype=torch.uint8, device="cuda")
    got_plan = _plan(n, K, d, 1, ws.numel())
    assert (got_plan[0], got_plan[2]) == (form, parts)
    P = B.norm_partials_per_row(p)
    xn, xl, part, part_l = torch.zeros_like(x), torch.zeros_like(x), *(torch.zeros((P, n, 2), device="cuda") for _ in range(2))
    B.dash_wo_residual_rownorm(p, a, w, x, n, xn, part, None, ws)
    B.dash_wo_residual_rownorm(p, a, w, x, n, xl, part_l, None, None)
    want = a.double() @ w.double()
    assert float((part - part_l).abs().max()) <= 1e-5 * float(part_l.abs().max())
    assert float((xn.double() - xl.double()).norm()) <= 1e-3 * float(xl.double().norm())
    full = x.double() + want
    assert bool(((xn.double() - full).abs() <= 2.0 ** -8 * full.abs() + 1e-5 * float(want.abs().max())).all())
    for e, t in ((0, want), (1, x.double())):
        blocks = torch.nn.functional.pad(t, (0, P * 256 - d)).reshape(n, P, 256).pow(2).sum(dim=2).t()
        assert float((part[..., e].double() - blocks).abs().max()) <= 1e-4 * float(blocks.max())


# rows, width, heads of 64, key/value heads, feed-forward width: the forms of the q/k/v product over the concatenated weight, of the one over
# w_q (plain store), of gate and up, and of the down projection
FRONT_AND_FFN = {(70, 512, 6, 2, 704): (16, 16, 16, 16), (333, 1024, 8, 4, 1408): (32, 16, 1, 32), (1205, 512, 12, 2, 1472): (1, 0, 2, 0),
                 (2300, 512, 8, 2, 2816): (1, 1, -1, 1), (149, 64, 52, 2, 1664): (0, 0, 0, 16), (1205, 512, 40, 2, 2240): (2, 2, 3, 0),
                 (2000, 512, 36, 2, 1152): (3, 3, 3, 0), (900, 1024, 72, 4, 2816): (4, 4, 4, 0)}


@pytest.mark.parametrize("n,d,hq,hkv,m", FRONT_AND_FFN)
def test_forms_of_front_end_and_feed_forward(n, d, hq, hkv, m):
    p = B.make_params(d, hq, hkv, 64, rule=B.RULE_NONE)
    qkv, ffn = max(B.qkv_workspace_bytes(p, n), 256), B.ffn_workspace_bytes(p, n, m)
    up256 = lambda v: -(-v // 256) * 256
    ffn -= up256(n * d * 2) + up256(n * m * 2) + up256(n * B.norm_partials_per_row(p) * 8)  # what is left for the products
    got = [_plan(n, d, N, 0, qkv)[0] for N in ((hq + 2 * hkv) * 64, hq * 64)] + [_plan(n, d, 2 * m, 0, ffn)[0], _plan(n, m, d, 0, ffn)[0]]
    assert tuple(got) == FRONT_AND_FFN[n, d, hq, hkv, m]


@pytest.mark.parametrize("n,d,hq,hkv,m", FRONT_AND_FFN)
def test_front_end_and_feed_forward(n, d, hq, hkv, m):
    """The q/k/v routing, plain store and gating epilogues at rows and widths that end inside tiles. h is rounded to bf16 on
    the way as the library does it; results carry one bf16 rounding of a sum of d (or m) products."""
    rng = np.random.default_rng(n)
    dh = 64
    p = B.make_params(d, hq, hkv, dh, rule=B.RULE_NONE)
    x, w = _rand(rng, (n, d), 2.0), _rand(rng, (d, (hq + 2 * hkv) * dh), d ** -0.5)
    ws = torch.empty((max(B.qkv_workspace_bytes(p, n), 256),), dtype=torch.uint8, device="cuda")
    h = torch.empty_like(x)
    new = lambda heads: torch.empty((n, heads, dh), dtype=torch.bfloat16, device="cuda")
    q, k, v = new(hq), new(hkv), new(hkv)
    B.dash_rmsnorm_qkv_fused(p, x, w, n, q, k, v, h, ws)
    parts = [t.contiguous() for t in w.split([hq * dh, hkv * dh, hkv * dh], dim=1)]
    q2, k2, v2 = new(hq), new(hkv), new(hkv)
    B.dash_rmsnorm_qkv(p, x, *parts, n, q2, k2, v2, torch.empty_like(x), ws)
    xd = x.double()
    hd = (xd * torch.rsqrt(xd.pow(2).mean(dim=1, keepdim=True) + 1e-6)).bfloat16().double()
    for got, wt in ((q, parts[0]), (k, parts[1]), (v, parts[2]), (q2, parts[0]), (k2, parts[1]), (v2, parts[2])):
        want = hd @ wt.double()
        # a row norm whose last fp32 bit differs may move a few of a row's h by one bf16 step: 2-norm, not elements
        assert float((got.reshape(n, -1).double() - want).norm() / want.norm()) <= 4e-3
    gate, up, down = _rand(rng, (d, m), d ** -0.5), _rand(rng, (d, m), d ** -0.5), _rand(rng, (m, d), m ** -0.5)
    out = torch.empty_like(x)
    fws = torch.empty((B.ffn_workspace_bytes(p, n, m),), dtype=torch.uint8, device="cuda")
    B.dash_ffn_swiglu(p, x, B.interleave_gate_up(gate, up), down, n, m, out, fws)
    act = (torch.nn.functional.silu(hd @ gate.double()) * (hd @ up.double())).bfloat16().double()
    upd = act @ down.double()
    assert float((out.double() - xd - upd).abs().max()) <= 2.0 ** -8 * float((xd + upd).abs().max()) + 4e-3 * float(upd.abs().max())


def _rest_parts(M, K, N, scratch):
    lib = _lib()
    lib.dash_rest_parts.argtypes = [ctypes.c_int] * 4 + [ctypes.c_ulonglong]
    return lib.dash_rest_parts(M, K, N, torch.cuda.get_device_properties(0).multi_processor_count, scratch)


@pytest.mark.parametrize("n,K,d", [(4617, 3584, 3584), (4900, 3584, 3400)])
def test_left_over_tiles_in_k_parts_projection(n, K, d):
    """Products whose few left-over half tiles are cut along K (the last row tile holds 9 and 36 rows; the last column tile
    whole and 72 columns): x_next and norms as in test_projection."""
    rng = np.random.default_rng(n)
    a, w, x = _rand(rng, (n, K)), _rand(rng, (K, d), K ** -0.5), _rand(rng, (n, d), 3.0)
    p = B.make_params(d, K // 64, 1, 64, rule=B.RULE_NONE)
    ws = torch.empty((64 << 20,), dtype=torch.uint8, device="cuda")
    assert _plan(n, K, d, 1, ws.numel())[0] < 0 and _rest_parts(n, K, d, ws.numel()) > 1
    P = B.norm_partials_per_row(p)
    xn, part = torch.zeros_like(x), torch.zeros((P, n, 2), device="cuda")
    B.dash_wo_residual_rownorm(p, a, w, x, n, xn, part, None, ws)
    want = a.double() @ w.double()
    full = x.double() + want
    assert bool(((xn.double() - full).abs() <= 2.0 ** -8 * full.abs() + 1e-5 * float(want.abs().max())).all())
    for e, t in ((0, want), (1, x.double())):
        blocks = torch.nn.functional.pad(t, (0, P * 256 - d)).reshape(n, P, 256).pow(2).sum(dim=2).t()
        assert float((part[..., e].double() - blocks).abs().max()) <= 1e-4 * float(blocks.max())


def test_left_over_tiles_in_k_parts_front_end_and_feed_forward():
    """The routing, store and gating epilogues of the second pass, and a long contraction."""
    rng = np.random.default_rng(3)
    d, hq, hkv, dh = 3584, 28, 4, 128
    p = B.make_params(d, hq, hkv, dh, rule=B.RULE_NONE)
    for n, fused in ((3612, True), (4617, False)):
        x, w = _rand(rng, (n, d), 2.0), _rand(rng, (d, (hq + 2 * hkv) * dh), d ** -0.5)
        ws = torch.empty((B.qkv_workspace_bytes(p, n),), dtype=torch.uint8, device="cuda")
        assert _rest_parts(n, d, 4608 if fused else 3584, ws.numel()) > 1
        q, k, v = (torch.zeros((n, h, dh), dtype=torch.bfloat16, device="cuda") for h in (hq, hkv, hkv))
        parts = [t.contiguous() for t in w.split([hq * dh, hkv * dh, hkv * dh], dim=1)]
        if fused:
            B.dash_rmsnorm_qkv_fused(p, x, w, n, q, k, v, torch.empty_like(x), ws)
        else:
            B.dash_rmsnorm_qkv(p, x, *parts, n, q, k, v, torch.empty_like(x), ws)
        hd = (x.double() * torch.rsqrt(x.double().pow(2).mean(dim=1, keepdim=True) + 1e-6)).bfloat16().double()
        for got, wt in zip((q, k, v), parts):
            want = hd @ wt.double()
            row = (got.reshape(n, -1).double() - want).norm(dim=1) / want.norm(dim=1)
            assert float(row.max()) <= 4e-3
    n, m = 400, 18944
    x = _rand(rng, (n, d), 2.0)
    gate, up, down = _rand(rng, (d, m), d ** -0.5), _rand(rng, (d, m), d ** -0.5), _rand(rng, (m, d), m ** -0.5)
    fws = torch.empty((B.ffn_workspace_bytes(p, n, m),), dtype=torch.uint8, device="cuda")
    out = torch.empty_like(x)
    B.dash_ffn_swiglu(p, x, B.interleave_gate_up(gate, up), down, n, m, out, fws)
    xd = x.double()
    hd = (xd * torch.rsqrt(xd.pow(2).mean(dim=1, keepdim=True) + 1e-6)).bfloat16().double()
    act = (torch.nn.functional.silu(hd @ gate.double()) * (hd @ up.double())).bfloat16().double()
    upd = act @ down.double()
    assert float((out.double() - xd - upd).abs().max()) <= 2.0 ** -8 * float((xd + upd).abs().max()) + 4e-3 * float(upd.abs().max())
