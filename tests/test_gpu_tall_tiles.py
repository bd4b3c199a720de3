"""The 192 x 128 small-tile product with the residual and norm and the q/k/v epilogues, rows and columns ending inside tiles, against fp64;
plain store and gating: test_gpu_small_tiles.FRONT_AND_FFN."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2604_18103_amd import binding as B
from test_gpu_small_tiles import _rand
from test_tall_tile_plan import TALL, tall_plan

pytestmark = pytest.mark.gpu


def _units():
    return torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("n,heads,d", [(1153, 16, 3584), (1345, 17, 3592), (1663, 18, 3400), (1728, 56, 3584), (4609, 16, 1160)])
def test_projection(n, heads, d):
    """One bf16 rounding of the result (at most 2^-8 of the element) beside fp32 sums of K products (1e-5 of the largest); norms: fp32 sums
    of d squares in any order, 1e-4."""
    K, rng = heads * 64, np.random.default_rng(n)
    a, w, x = _rand(rng, (n, K)), _rand(rng, (K, d), K ** -0.5), _rand(rng, (n, d), 3.0)
    p = B.make_params(d, heads, 1, 64, rule=B.RULE_NONE)
    ws = torch.empty((64 << 20,), dtype=torch.uint8, device="cuda")
    assert tall_plan(n, K, d, _units(), 1, ws.numel())[0] == TALL
    xn, part = torch.zeros_like(x), torch.zeros((B.norm_partials_per_row(p), n, 2), device="cuda")
    B.dash_wo_residual_rownorm(p, a, w, x, n, xn, part, None, ws)
    want = a.double() @ w.double()
    full = x.double() + want
    assert bool(((xn.double() - full).abs() <= 2.0 ** -8 * full.abs() + 1e-5 * float(want.abs().max())).all())
    total = part.double().sum(dim=0)
    for e, t in ((0, want), (1, x.double())):
        assert bool(((total[:, e] - t.pow(2).sum(dim=1)).abs() <= 1e-4 * t.pow(2).sum(dim=1)).all())


@pytest.mark.parametrize("n,d,hq,hkv,dh", [(1200, 1024, 28, 4, 128), (3001, 1024, 16, 4, 64), (1345, 1088, 52, 2, 64)])
@pytest.mark.parametrize("rotate", [False, True])
def test_front_end(n, d, hq, hkv, dh, rotate):
    """h is rounded to bf16 on the way as the library does it; results carry one bf16 rounding (1.7e-3 of a row in the 2-norm, bound 4e-3)."""
    rng, N = np.random.default_rng(n), (hq + 2 * hkv) * dh
    assert tall_plan(n, d, N, _units(), 0, 64 << 20)[0] == TALL
    x, w = _rand(rng, (n, d), 3.0), _rand(rng, (d, N), d ** -0.5)
    idx = torch.arange(3, n + 3, dtype=torch.int32, device="cuda")
    p = B.make_params(d, hq, hkv, dh, rule=B.RULE_NONE)
    q, k, v = (torch.zeros((n, h, dh), dtype=torch.bfloat16, device="cuda") for h in (hq, hkv, hkv))
    h, ws = torch.empty_like(x), torch.empty((64 << 20,), dtype=torch.uint8, device="cuda")
    if rotate:
        B.dash_rmsnorm_qkv_rope(p, x, w, idx, n, 1e6, q, k, v, h, ws)
    else:
        B.dash_rmsnorm_qkv_fused(p, x, w, n, q, k, v, h, ws)
    xd = x.double()
    hd = (xd * torch.rsqrt(xd.pow(2).mean(dim=1, keepdim=True) + 1e-6)).bfloat16().double()
    want = (hd @ w.double()).reshape(n, hq + 2 * hkv, dh)
    if rotate:
        half = dh // 2
        ang = idx.double()[:, None] * 1e6 ** (-torch.arange(half, device="cuda", dtype=torch.float64) / half)
        c, s = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
        lo, hi = want[:, :hq + hkv, :half].clone(), want[:, :hq + hkv, half:].clone()
        want[:, :hq + hkv, :half], want[:, :hq + hkv, half:] = lo * c - hi * s, lo * s + hi * c
    got = torch.cat([q, k, v], dim=1).double()
    assert float(((got - want).norm(dim=2) / want.norm(dim=2)).max()) <= 4e-3
