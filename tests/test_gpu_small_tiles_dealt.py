"""The 128 x 128 small-tile product with dealt-out requests on contractions of fewer, as many and a few more K steps than it has
operand stages, rows and columns ending inside tiles, against fp64."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2604_18103_amd import binding as B
from test_gpu_small_tiles import _plan, _rand

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,steps,d", [(2201, 1, 1520), (1207, 2, 2800), (1108, 3, 3520), (4021, 4, 1000), (628, 5, 4512), (856, 6, 3200)])
def test_few_steps(n, steps, d):
    """One bf16 rounding of the result (at most 2^-8 of the element) beside fp32 sums of K products (1e-5 of the largest)."""
    K, rng = 64 * steps, np.random.default_rng(n)
    a, w, x = _rand(rng, (n, K)), _rand(rng, (K, d), K ** -0.5), _rand(rng, (n, d), 3.0)
    p = B.make_params(d, steps, 1, 64, rule=B.RULE_NONE)
    ws = torch.empty((64 << 20,), dtype=torch.uint8, device="cuda")
    assert _plan(n, K, d, 1, ws.numel())[:3:2] == (2, 1)
    xn, part = torch.zeros_like(x), torch.zeros((B.norm_partials_per_row(p), n, 2), device="cuda")
    B.dash_wo_residual_rownorm(p, a, w, x, n, xn, part, None, ws)
    want = a.double() @ w.double()
    full = x.double() + want
    assert bool(((xn.double() - full).abs() <= 2.0 ** -8 * full.abs() + 1e-5 * float(want.abs().max())).all())
    total = part.double().sum(dim=0)
    assert bool(((total[:, 0] - want.pow(2).sum(dim=1)).abs() <= 1e-4 * want.pow(2).sum(dim=1)).all())
