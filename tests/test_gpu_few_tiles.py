"""The product on the tiles for the fewest rows: rows and columns ending inside tiles, waves without a K step, with one and with several, K
parts, and every epilogue, against fp64."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2604_18103_amd import binding as B
from test_few_tile_plan import few_plan
from test_gpu_small_tiles import _rand

pytestmark = pytest.mark.gpu


def _units():
    return torch.cuda.get_device_properties(0).multi_processor_count


# (rows, K steps, width, rows of a tile, K parts)
@pytest.mark.parametrize("n,steps,d,bm,parts", [(1, 1, 64, 16, 1), (15, 7, 200, 16, 1), (17, 8, 512, 16, 1), (33, 9, 1032, 16, 1), (16, 56, 3584, 16, 4),
                                                (33, 16, 3584, 16, 1), (31, 56, 3584, 32, 4), (333, 16, 1024, 32, 1), (45, 56, 3584, 48, 4),
                                                (177, 56, 3584, 48, 1), (145, 20, 4096, 48, 1), (700, 8, 520, 32, 1), (1000, 5, 640, 48, 1)])
def test_projection(n, steps, d, bm, parts):
    """x_next: one bf16 rounding (2^-8 of the element covers a sum on the other side of a tie) beside fp32 sums of K products (1e-5 of
    the largest); norms: fp32 sums of d squares, 1e-4."""
    K, rng = 64 * steps, np.random.default_rng(n + d)
    a, w, x = _rand(rng, (n, K)), _rand(rng, (K, d), K ** -0.5), _rand(rng, (n, d), 3.0)
    p = B.make_params(d, steps, 1, 64, rule=B.RULE_NONE)
    ws = torch.empty((64 << 20,), dtype=torch.uint8, device="cuda")
    assert few_plan(n, K, d, _units(), scratch=ws.numel())[::2] == (bm, parts)
    xn, part = torch.zeros_like(x), torch.zeros((B.norm_partials_per_row(p), n, 2), device="cuda")
    B.dash_wo_residual_rownorm(p, a, w, x, n, xn, part, None, ws)
    want = a.double() @ w.double()
    full = x.double() + want
    assert bool(((xn.double() - full).abs() <= 2.0 ** -8 * full.abs() + 1e-5 * float(want.abs().max())).all())
    for e, t in ((0, want), (1, x.double())):
        blocks = torch.nn.functional.pad(t, (0, part.shape[0] * 256 - d)).reshape(n, -1, 256).pow(2).sum(dim=2).t()
        assert float((part[..., e].double() - blocks).abs().max()) <= 1e-4 * float(blocks.max())


@pytest.mark.parametrize("n", [1, 47, 177, 300])
def test_front_end_with_heads_of_64_and_feed_forward(n):
    """q/k/v routing with the rotary embedding, gating and the residual: the same calls without scratch take the large tiles, whose sums
    differ in their order only (one bf16 step, 2^-7, of an element that rounds the other way, 1e-3 over all; the feed-forward's
    gated product is rounded in between)."""
    rng, d, hq, hkv, m = np.random.default_rng(n), 1024, 16, 4, 2816
    x, w = _rand(rng, (n, d), 2.0), _rand(rng, (d, (hq + 2 * hkv) * 64), d ** -0.5)
    idx = torch.arange(0, 3 * n, 3, dtype=torch.int32, device="cuda")
    p = B.make_params(d, hq, hkv, 64)
    ws = torch.empty((64 << 20,), dtype=torch.uint8, device="cuda")
    assert few_plan(n, d, w.shape[1], _units(), norms=0, head=64)[0] > 0
    out = []
    for scratch in (ws, None):
        q, k, v, h = torch.empty((n, hq, 64), dtype=x.dtype, device="cuda"), *(torch.empty((n, hkv, 64), dtype=x.dtype, device="cuda") for _ in range(2)), torch.empty_like(x)
        B.dash_rmsnorm_qkv_rope(p, x, w, idx, n, 1e6, q, k, v, h, scratch)
        out.append(torch.cat([t.reshape(n, -1) for t in (q, k, v)], dim=1).double())
    assert float((out[0] - out[1]).norm()) <= 4e-3 * float(out[1].norm())  # without scratch the rotation works on rounded q and k
    gate, up, down = _rand(rng, (d, m), d ** -0.5), _rand(rng, (d, m), d ** -0.5), _rand(rng, (m, d), m ** -0.5)
    y = torch.empty_like(x)
    fws = torch.empty((B.ffn_workspace_bytes(p, n, m),), dtype=torch.uint8, device="cuda")
    B.dash_ffn_swiglu(p, x, B.interleave_gate_up(gate, up), down, n, m, y, fws)
    xd = x.double()
    h = (xd * torch.rsqrt((xd * xd).mean(dim=1, keepdim=True) + 1e-6)).bfloat16().double()
    g = (torch.nn.functional.silu(h @ gate.double()) * (h @ up.double())).bfloat16().double()
    want = xd + g @ down.double()
    assert float((y.double() - want).norm()) <= 4e-3 * float(want.norm())
