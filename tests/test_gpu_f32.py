"""The fp32 attention and projection kernels at the edges of their tiles, against the fp64 oracle."""
import numpy as np
import pytest
import torch

from oracle import reference as ref
from paper_2604_18103_amd import binding as B

pytestmark = pytest.mark.gpu


def _attention(n, hq, hkv, dh, causal, seed, v_edit=None):
    rng = np.random.default_rng(seed)
    q, k, v = (rng.standard_normal((n, h, dh)).astype(np.float32) for h in (hq, hkv, hkv))
    pos = np.sort(rng.permutation(3 * n + 1)[:n]).astype(np.int32)
    if v_edit is not None:
        v_edit(v)
    p = B.make_params(hq * dh, hq, hkv, dh, dtype=B.DASH_F32, causal=causal)
    dev = [torch.from_numpy(a).cuda() for a in (q, k, v, pos)]
    o = torch.empty((n, hq * dh), dtype=torch.float32, device="cuda")
    B.dash_flash_fwd(p, *dev[:3], dev[3], n, o)
    return q, k, v, pos, o.cpu().numpy()


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 33, 255, 257, 530])
def test_f32_attention_tile_edges(n, dh):
    """16-row tiles, 32-key blocks dealt to 8 waves: lengths around each, causal and not. Sums of n + head_dim fp32
    terms: 1e-5 of the row's largest element is above ten times the measured error (3e-7 in the 2-norm)."""
    for causal in (True, False):
        q, k, v, pos, o = _attention(n, 4, 2, dh, causal, seed=n + dh)
        want = ref.attention_rows(q, k, v, pos, causal=causal)
        err = np.abs(o - want).max(axis=1) / np.abs(want).max(axis=1)
        assert err.max() <= 1e-5, (n, dh, causal, err.max())


def test_f32_attention_reads_nothing_that_a_row_does_not_see():
    """An infinite and a NaN value in a later row of the same key block leave the earlier rows untouched."""
    bad = 40

    def edit(v):
        v[bad, :, 3] = np.inf
        v[bad, :, 70] = np.nan

    q, k, v, pos, o = _attention(75, 2, 1, 128, True, seed=5, v_edit=edit)
    want = ref.attention_rows(q[:bad], k[:bad], v[:bad], pos[:bad], causal=True)
    assert np.abs(o[:bad] - want).max() <= 1e-5 * np.abs(want).max()
    assert not np.isfinite(o[bad:, 3]).any() and np.isnan(o[bad:, 70]).all()
    assert np.isfinite(o[bad:, 4]).all()


@pytest.mark.parametrize("n,hq,dh,d", [(1, 1, 64, 4), (31, 4, 64, 100), (33, 1, 128, 68), (70, 2, 128, 260)])
def test_f32_projection_tile_edges(n, hq, dh, d):
    """32 x 64 tiles, K in chunks of 16 over 8 waves (4, 16, 8 and 16 chunks here); widths that end inside a tile.
    Sums of K fp32 products, K <= 256: 1e-5 of the row's largest element."""
    rng = np.random.default_rng(d)
    K = hq * dh
    a, w, x = (rng.standard_normal(s).astype(np.float32) for s in ((n, K), (K, d), (n, d)))
    p = B.make_params(d, hq, 1, dh, dtype=B.DASH_F32)
    P = B.norm_partials_per_row(p)
    xn, delta = (torch.empty((n, d), dtype=torch.float32, device="cuda") for _ in range(2))
    part = torch.empty((P, n, 2), dtype=torch.float32, device="cuda")
    ta, tw, tx = (torch.from_numpy(t).cuda() for t in (a, w, x))
    B.dash_wo_residual_rownorm(p, ta, tw, tx, n, xn, part, delta, None)
    want = ref.project(a, w)
    scale = np.abs(want).max(axis=1, keepdims=True)
    assert np.abs(delta.cpu().numpy() - want).max() <= 1e-5 * scale.max()
    assert np.abs(xn.cpu().numpy() - (x + want)).max() <= 1e-5 * np.abs(x + want).max()
    sums = part.cpu().numpy().astype(np.float64).sum(axis=0)
    np.testing.assert_allclose(sums[:, 0], (want ** 2).sum(axis=1), rtol=1e-5)
    np.testing.assert_allclose(sums[:, 1], (x.astype(np.float64) ** 2).sum(axis=1), rtol=1e-5)


def test_f32_projection_of_more_rows_than_a_grid_dimension_holds_tiles():
    """2.1 million rows are 65628 row tiles of 32, beyond the 65535 workgroups that a launch has along y."""
    n, K, d = 2_100_077, 64, 4
    g = torch.Generator(device="cuda").manual_seed(2)
    a, w, x = (torch.randn(s, generator=g, device="cuda") for s in ((n, K), (K, d), (n, d)))
    p = B.make_params(d, 1, 1, 64, dtype=B.DASH_F32)
    xn, part = torch.zeros_like(x), torch.zeros((1, n, 2), device="cuda")
    B.dash_wo_residual_rownorm(p, a, w, x, n, xn, part)
    want = a.double() @ w.double()
    assert float((xn.double() - x.double() - want).abs().max()) <= 1e-5 * float(want.abs().max())
    assert float((part[0, :, 0].double() - want.pow(2).sum(dim=1)).abs().max()) <= 1e-5 * float(want.pow(2).sum(dim=1).max())
    assert float((part[0, :, 1].double() - x.double().pow(2).sum(dim=1)).abs().max()) <= 1e-5 * float(x.pow(2).sum(dim=1).max())
