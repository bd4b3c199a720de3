"""The bf16 attention's few-row form (32 query rows per workgroup, keys split over its waves) at the edges of its blocks, and the
two-group form of the tiled kernel at lengths beyond that form's range, against the fp64 oracle."""
import numpy as np
import pytest
import torch

from oracle import reference as ref
from paper_2604_18103_amd import binding as B
from test_attention_form import ONE_AND_TAIL, TWO
from test_gpu_attention_groups import _run
from test_gpu_infinite_keys import _attention
from test_staging_addresses import _load

pytestmark = pytest.mark.gpu


def _units():
    return torch.cuda.get_device_properties(0).multi_processor_count


# eight waves (few workgroups) and four; one block, one per wave, one more than the waves, remainders of 1 and 31 rows
@pytest.mark.parametrize("hq,hkv,dh", [(4, 2, 128), (4, 2, 64), (40, 8, 128), (80, 8, 64)])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 63, 65, 128, 129, 223, 256, 257, 289])
def test_block_edges(n, hq, hkv, dh):
    waves = 8 if -(-n // 32) * hq <= _units() * (2 if dh == 64 else 1) else 4
    for causal in (1, 0):
        took = _load().dash_few_waves(n, hq, dh, causal, _units())
        assert took in (waves, 0) and (took or not causal)
        _run(n, hq, hkv, dh, bool(causal), seed=n + dh)


@pytest.mark.parametrize("n,hq,hkv,dh,causal", [(40, 4, 2, 64, True), (64, 4, 2, 64, True), (128, 4, 2, 128, True), (130, 4, 2, 128, False),
                                                (193, 4, 2, 64, True), (321, 28, 4, 128, True), (177, 28, 4, 128, True), (333, 4, 2, 128, False),
                                                (800, 28, 4, 128, True), (1000, 16, 4, 64, True), (2500, 16, 4, 64, True), (500, 28, 4, 128, False)])
def test_ordinary_rows_closely(n, hq, hkv, dh, causal):
    """P and the result are rounded to bf16 (each 1.6e-3 of a row in the 2-norm, test_gpu_attention_groups), Q is not rounded
    again: 2.3e-3, bound 3e-3 on the mean; a row that few keys carry has fewer independent roundings, 8e-3 on the largest."""
    assert _load().dash_few_waves(n, hq, dh, int(causal), _units()) in (4, 8)
    rng = np.random.default_rng(n)
    q, k, v = (torch.from_numpy(rng.standard_normal((n, h, dh)).astype(np.float32)).bfloat16() for h in (hq, hkv, hkv))
    pos = np.sort(rng.permutation(2 * n + 1)[:n]).astype(np.int32)
    p = B.make_params(hq * dh, hq, hkv, dh, causal=causal)
    o = torch.full((n + 1, hq * dh), 7.0, dtype=torch.bfloat16, device="cuda")
    B.dash_flash_fwd(p, q.cuda(), k.cuda(), v.cuda(), torch.from_numpy(pos).cuda(), n, o)
    assert bool((o[n] == 7.0).all())  # nothing beyond the last row
    rows = np.unique(np.r_[0:min(n, 8), rng.integers(0, n, 40), n - 1])
    want = ref.attention_rows(*(t.float().numpy() for t in (q, k, v)), pos, rows=rows, causal=causal).reshape(len(rows), hq, dh)
    got = o.float().cpu().numpy()[rows].reshape(len(rows), hq, dh)
    err = np.linalg.norm(got - want, axis=2) / np.linalg.norm(want, axis=2)
    assert float(err.max()) <= 8e-3 and float(err.mean()) <= 3e-3


@pytest.mark.parametrize("low", [False, True])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dh", [64, 128])
def test_blocks_of_infinite_keys(dh, causal, low):
    """A wave's first block without a finite score, its second, all of one wave's, in workgroups of four waves and eight."""
    for n, hq in ((330, 4), (330, 48 if causal else 24)):
        for infinite in (slice(0, 32), slice(32, 64), slice(128, 192), slice(0, 290)):
            _attention(n, hq, 2, dh, causal, infinite, low, np.arange(0, n, 3))


@pytest.mark.parametrize("n,hq,hkv,dh,causal", [(897, 28, 4, 128, True), (960, 28, 4, 128, True), (1023, 28, 4, 128, True), (1025, 28, 4, 128, True),
                                                (2561, 16, 4, 64, True), (2625, 16, 4, 64, True), (2752, 16, 4, 64, True),
                                                (641, 28, 4, 128, False), (703, 28, 4, 128, False), (1153, 16, 4, 64, False), (1217, 16, 4, 64, False)])
def test_two_key_groups_beyond_it(n, hq, hkv, dh, causal):
    """128-row workgroups of the tiled kernel whose last tile holds 1 to 128 rows, with an odd and an even number of key tiles;
    and without a finite score a first key tile of either group, and the first two of group 1."""
    lib = _load()
    assert lib.dash_few_waves(n, hq, dh, int(causal), _units()) == 0 and lib.dash_fa_form(n, hq, dh, int(causal), _units()) == TWO
    rows = np.unique(np.r_[0, 1, 63, 64, 127, 128, n // 2, n - 66, n - 65, n - 2, n - 1])
    _run(n, hq, hkv, dh, causal, seed=n, rows=rows)
    for infinite in (slice(64, 128), slice(0, 64), slice(64, 256)):
        _attention(n, hq, hkv, dh, causal, infinite, n % 2 == 1, rows)


@pytest.mark.parametrize("n,hq,hkv,dh,few", [(4129, 16, 4, 64, 1), (4351, 16, 4, 64, 1), (2336, 28, 4, 128, 1), (2559, 28, 4, 128, 1), (1279, 64, 8, 128, 0)])
def test_the_rows_beyond_the_last_whole_tile(n, hq, hkv, dh, few):
    """Without a causal mask, 32, 33 and 255 of them, in the few-row form and, where its workgroups would not all be resident, in the split one."""
    lib = _load()
    assert lib.dash_fa_form(n, hq, dh, 0, _units()) == ONE_AND_TAIL and lib.dash_fa_few_tail(n, hq, dh, _units()) == few
    end = n - n % 256
    _run(n, hq, hkv, dh, False, seed=n, rows=np.unique(np.r_[0, end - 1, end, end + 1, min(end + 31, n - 1), min(end + 32, n - 1), n - 2, n - 1]))
