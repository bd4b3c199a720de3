"""Products whose last round runs on 192- or 224-row tiles, every epilogue, against fp64 sums of the same bf16 operands and against
the calls without scratch."""
import pytest
import torch

from paper_2604_18103_amd import binding as B
from test_gpu_rope_epilogue import test_against_fp64 as _rope
from test_gpu_small_tiles import _rand, test_front_end_and_feed_forward as _front_and_ffn
from test_row_plan import _plan
import numpy as np

pytestmark = pytest.mark.gpu


# rows, heads of 64, width, 16-row blocks per wave, 256-row row tiles before them; last row tiles of 1, 16 and 17 rows and whole ones
@pytest.mark.parametrize("n,heads,d,rb,whole", [(2497, 56, 3584, 6, 0), (2512, 56, 3584, 6, 0), (3456, 16, 3584, 6, 0), (3585, 16, 3584, 7, 0),
                                                (3601, 8, 3400, 7, 0), (7501, 296, 3584, 6, 18), (8193, 296, 3584, 7, 18)])
def test_projection(n, heads, d, rb, whole):
    """Bounds as for the small tiles (one bf16 rounding beside fp32 sums of K products, norms 1e-4); with and without the debug
    output the same bits."""
    K, rng = heads * 64, np.random.default_rng(n)
    assert _plan(n, K, d) == (rb, whole)
    a, w, x = _rand(rng, (n, K)), _rand(rng, (K, d), K ** -0.5), _rand(rng, (n, d), 3.0)
    p = B.make_params(d, heads, 1, 64, rule=B.RULE_NONE)
    ws = torch.empty((64 << 20,), dtype=torch.uint8, device="cuda")
    P = B.norm_partials_per_row(p)
    xn, part = torch.zeros_like(x), torch.zeros((P, n, 2), device="cuda")
    B.dash_wo_residual_rownorm(p, a, w, x, n, xn, part, None, ws)
    x2, part2, delta = torch.zeros_like(x), torch.zeros_like(part), torch.zeros((n, d), device="cuda")
    B.dash_wo_residual_rownorm(p, a, w, x, n, x2, part2, delta, None)
    assert torch.equal(xn.view(torch.int16), x2.view(torch.int16)) and torch.equal(part, part2)
    want = a.double() @ w.double()
    assert float((delta.double() - want).abs().max()) <= 1e-5 * float(want.abs().max()) * max(1.0, (K / 4096) ** 0.5)
    full = x.double() + want
    assert bool(((xn.double() - full).abs() <= 2.0 ** -8 * full.abs() + 2e-5 * float(want.abs().max())).all())
    for e, t in ((0, want), (1, x.double())):
        blocks = torch.nn.functional.pad(t, (0, P * 256 - d)).reshape(n, P, 256).pow(2).sum(dim=2).t()
        assert float((part[..., e].double() - blocks).abs().max()) <= 1e-4 * float(blocks.max())


def test_the_other_epilogues():
    """Routing, store and gating (28 column tiles), rotation at both head sizes, on 192 and 224 rows."""
    for n, rb in ((1701, 6), (1801, 7)):
        assert _plan(n, 512, 7168) == (rb, 0)
        _front_and_ffn(n, 512, 96, 8, 3584)
        for hq, hkv, dh in ((96, 8, 64), (48, 4, 128)):
            _rope(n, 512, hq, hkv, dh)
