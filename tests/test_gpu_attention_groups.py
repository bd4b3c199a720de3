"""The tiled bf16 attention kernel's two forms (one key group per workgroup, two for shorter sequences) at the edges of their
tiles, against the fp64 oracle; the shortest lengths, at the same edges, take the few-row form (test_gpu_attention_few)."""
import numpy as np
import pytest
import torch

from oracle import reference as ref
from paper_2604_18103_amd import binding as B
from test_attention_form import ONE, ONE_AND_TAIL, TWO
from test_staging_addresses import _load

pytestmark = pytest.mark.gpu


def _run(n, hq, hkv, dh, causal, seed, rows=None):
    rng = np.random.default_rng(seed)
    q, k, v = (torch.from_numpy(rng.standard_normal((n, h, dh)).astype(np.float32)).bfloat16() for h in (hq, hkv, hkv))
    # keys in either group's tiles that lift the softmax reference late in the sequence
    for row, f in ((70, 3.0), (130, 6.0), (n - 1, 5.0)):
        if row < n:
            k[row] *= f
    pos = np.sort(rng.permutation(2 * n + 1)[:n]).astype(np.int32)
    p = B.make_params(hq * dh, hq, hkv, dh, causal=causal)
    o = torch.empty((n, hq * dh), dtype=torch.bfloat16, device="cuda")
    B.dash_flash_fwd(p, q.cuda(), k.cuda(), v.cuda(), torch.from_numpy(pos).cuda(), n, o)
    want = ref.attention_rows(*(t.float().numpy() for t in (q, k, v)), pos, rows=rows, causal=causal)
    got = o.float().cpu().numpy()
    got = got if rows is None else got[rows]
    # Q, P and O are rounded to bf16 (2^-9 each). The scores reach about 6 * 4.5 * log2(e) = 40 in the log2 domain, where
    # the rounding of Q (2^-9 per element, random over the head's 64 or 128 dims) moves a score by up to about 0.05.
    err = np.abs(got - want).max(axis=1) / np.abs(want).max(axis=1)
    assert np.isfinite(got).all() and err.max() <= 6e-2 and err.mean() <= 1e-2, (n, dh, causal, err.max(), err.mean())


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 96, 127, 128, 129, 192, 193, 257, 320])
def test_two_key_groups_at_tile_edges(n, dh):
    """Lengths at the edges of the two key groups' tiles that are so short that the few-row form takes them; the two groups themselves
    run in test_gpu_attention_few.test_two_key_groups_beyond_it."""
    units = torch.cuda.get_device_properties(0).multi_processor_count
    for causal in (True, False):
        assert _load().dash_few_waves(n, 4, dh, int(causal), units) > 0
        _run(n, 4, 2, dh, causal, seed=n + dh)


@pytest.mark.parametrize("n,hq,hkv,dh,causal", [(5377, 16, 4, 64, True), (2433, 28, 4, 128, True), (1409, 28, 4, 128, False),
                                                (4097, 16, 4, 64, False), (4224, 16, 4, 64, False), (2400, 32, 8, 128, False)])
def test_one_key_group_with_a_nearly_empty_last_tile(n, hq, hkv, dh, causal):
    """Lengths just past the split form's range whose last 256-row tile holds 1, 129 and 129 rows: waves beyond the end
    do nothing. Without a causal mask also lengths whose last 1, 128 and 96 rows run as a launch of their own."""
    _run(n, hq, hkv, dh, causal, seed=n, rows=np.array([0, 1, 31, 32, 255, 256, n // 2, n - 130, n - 2, n - 1]))


@pytest.mark.parametrize("n,hq,hkv,dh,causal,form", [
    (1000, 28, 4, 128, True, TWO), (2303, 28, 4, 128, True, TWO), (2561, 16, 4, 64, True, TWO), (5000, 16, 4, 64, True, TWO),
    (1153, 16, 4, 64, False, TWO), (4480, 16, 4, 64, False, TWO), (1150, 28, 4, 128, False, TWO), (2433, 28, 4, 128, True, ONE),
    (5377, 16, 4, 64, True, ONE), (4097, 16, 4, 64, False, ONE_AND_TAIL), (4224, 16, 4, 64, False, ONE_AND_TAIL),
    (2400, 28, 4, 128, False, ONE_AND_TAIL), (2305, 28, 4, 128, False, ONE_AND_TAIL), (2432, 28, 4, 128, False, ONE_AND_TAIL),
    (1279, 64, 8, 128, False, ONE_AND_TAIL)])
def test_ordinary_rows_closely(n, hq, hkv, dh, causal, form):
    """Normal q, k and v, every tiled form by name; ONE_AND_TAIL's last rows in the few-row form, with 64 heads in the split one.
    A bf16 number has 8 significant bits: its rounding is uniform in +-2^-8 of the power of two below it, in the mean square
    2^-8 / sqrt(3) * 0.72 = 1.6e-3 of the number. Scores have unit variance, so Q's rounding moves a probability by that much, its
    own rounding again, and the result's a third time: 2.8e-3 of a row in the 2-norm, bound 3.5e-3 on the mean. A row that few
    keys carry has fewer independent roundings, each at most 3.9e-3: 8e-3 on the largest. A weight between the two groups that is
    off by a hundredth moves a row by about 7e-3, so the mean shows it."""
    units = torch.cuda.get_device_properties(0).multi_processor_count
    lib = _load()
    assert lib.dash_few_waves(n, hq, dh, int(causal), units) == 0 and lib.dash_fa_form(n, hq, dh, int(causal), units) == form
    assert form != ONE_AND_TAIL or lib.dash_fa_few_tail(n, hq, dh, units) == (hq != 64)
    rng = np.random.default_rng(n)
    q, k, v = (torch.from_numpy(rng.standard_normal((n, h, dh)).astype(np.float32)).bfloat16() for h in (hq, hkv, hkv))
    pos = np.sort(rng.permutation(2 * n + 1)[:n]).astype(np.int32)
    p = B.make_params(hq * dh, hq, hkv, dh, causal=causal)
    o = torch.empty((n, hq * dh), dtype=torch.bfloat16, device="cuda")
    B.dash_flash_fwd(p, q.cuda(), k.cuda(), v.cuda(), torch.from_numpy(pos).cuda(), n, o)
    rows = np.unique(np.r_[0:min(n, 8), rng.integers(0, n, 40), max(n - 130, 0), max(n - 65, 0), n - 1])
    want = ref.attention_rows(*(t.float().numpy() for t in (q, k, v)), pos, rows=rows, causal=causal).reshape(len(rows), hq, dh)
    got = o.float().cpu().numpy()[rows].reshape(len(rows), hq, dh)
    err = np.linalg.norm(got - want, axis=2) / np.linalg.norm(want, axis=2)
    top, mean = float(err.max()), float(err.mean())
    assert top <= 8e-3 and mean <= 3.5e-3
