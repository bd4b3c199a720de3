"""Attention over keys whose score is -inf for some rows: a whole key tile of them has no finite maximum to take the softmax
reference from, in the first tile of either key group. A row is finite wherever the fp64 oracle's is."""
import numpy as np
import pytest
import torch

from oracle import reference as ref
from paper_2604_18103_amd import binding as B
from test_staging_addresses import _load

pytestmark = pytest.mark.gpu


def _attention(n, hq, hkv, dh, causal, infinite, low, rows):
    rng = np.random.default_rng(n + dh)
    q, k, v = (torch.from_numpy(rng.standard_normal((n, h, dh)).astype(np.float32)).bfloat16() for h in (hq, hkv, hkv))
    q[:, :, 0] = -q[:, :, 0].abs() - 0.5
    q[5::16, :, 0] *= -1.0          # these rows score +inf against the infinite keys: NaN in the oracle too
    k[infinite, :, 0] = float("inf")
    if low:                         # every other score far below 0: a reference of 0 would leave no probability
        q[:, :, 1], k[:, :, 1] = 30.0, -60.0
    pos = np.arange(n, dtype=np.int32)
    p = B.make_params(hq * dh, hq, hkv, dh, causal=causal)
    o = torch.empty((n, hq * dh), dtype=torch.bfloat16, device="cuda")
    B.dash_flash_fwd(p, q.cuda(), k.cuda(), v.cuda(), torch.from_numpy(pos).cuda(), n, o)
    with np.errstate(all="ignore"):
        want = ref.attention_rows(*(t.float().numpy() for t in (q, k, v)), pos, rows=rows, causal=causal)
    got = o.float().cpu().numpy()[rows]
    fine = np.isfinite(want).all(axis=1)
    assert fine.any() and np.isfinite(got[fine]).all(), (n, dh, causal, low, rows[fine][~np.isfinite(got[fine]).all(axis=1)][:8])
    # The bounds of the attention tests: Q, P and O are rounded to bf16. With `low` the logits reach 1800 / sqrt(dh), and the
    # rounding of Q (2^-9 of its element) moves all of a row's logits by the same amount but for the keys' spread around it.
    err = np.abs(got[fine] - want[fine]).max(axis=1) / np.abs(want[fine]).max(axis=1)
    assert err.max() <= 6e-2 and err.mean() <= 1e-2, (n, dh, causal, low, err.max(), err.mean())


@pytest.mark.parametrize("low", [False, True])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dh", [64, 128])
def test_a_tile_of_infinite_keys(dh, causal, low):
    """So few rows that the few-row form takes them: whole key blocks of one to all of its waves. (The tiles of two key groups:
    test_gpu_attention_few.test_two_key_groups_beyond_it.)"""
    n = 330
    assert _load().dash_few_waves(n, 4, dh, int(causal), torch.cuda.get_device_properties(0).multi_processor_count) > 0
    for infinite in (slice(64, 128), slice(0, 64), slice(64, 256)):
        _attention(n, 4, 2, dh, causal, infinite, low, np.arange(n))


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("hq,hkv,dh,n", [(16, 4, 64, 5377), (28, 4, 128, 2433)])
def test_one_key_group(hq, hkv, dh, n, causal):
    """The first tile, and the first three, of 256-row workgroups; without a causal mask of 16 heads of 64 the first of group 0, and
    the first of group 1 beside the first two of group 0."""
    for infinite in (slice(0, 64), slice(0, 192)):
        _attention(n, hq, hkv, dh, causal, infinite, True, np.array([0, 63, 64, 191, 192, 200, 255, 256, 300, n // 2, n - 1]))
