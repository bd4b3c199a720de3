"""The one-launch TopK decision on scores that reach each of its ends: bins of one key value, a bin's last keys by counting, further
passes inside a crowded bin; cuts at every edge of a crowd; both directions; bit for bit against the oracle."""
import numpy as np
import pytest
import torch

from oracle import reference as ref
from paper_2604_18103_amd import binding as B

pytestmark = pytest.mark.gpu


def _steps(first, count):
    """`count` consecutive fp32 numbers from `first` on."""
    return (np.float32(first).view(np.uint32) + np.arange(count, dtype=np.uint32)).view(np.float32)


def _scores(kind, n, rng):
    if kind == "dense":            # all keys within 2048 of each other: a bin is one value
        return rng.choice(_steps(1.0, min(2000, n)), n)
    if kind == "crowd":            # 500 neighbours far inside a wide range: two passes more
        s = np.exp(rng.normal(0.0, 8.0, n))
        s[: min(n, 500)] = _steps(3.0, min(n, 500))
    elif kind == "tied crowd":     # the same with every value three times
        s = np.exp(rng.normal(0.0, 8.0, n))
        s[: min(n, 600)] = np.repeat(_steps(3.0, 200), 3)[: min(n, 600)]
    elif kind == "edge":           # scores from 0 to 256: bins of 2^20 keys, an eighth of an octave; 64 and 65 different keys in one each
        s = np.r_[0.0, 256.0, _steps(8.01, 64), _steps(16.01, 65), rng.uniform(64, 200, max(n - 131, 0))][:n]
        assert n < 131 or (len(np.unique(_steps(8.01, 64))), len(np.unique(_steps(16.01, 65)))) == (64, 65)
    elif kind == "outliers":       # a crowd of few values behind an outlier on either side: its own range is one value or few
        s = np.round(rng.normal(size=n) * 8) / 8
        s[: min(n, 2)] = (np.inf, -np.inf)[: min(n, 2)]
    elif kind == "top":            # the last bin of the whole range is crowded and ends with the largest key that there is
        s = rng.choice(_steps(3.0e38, 40), n)
        s[: n // 3], s[n // 3: n // 3 + 1] = np.nan, -np.inf
    else:                          # signed zeros, infinities, NaN, the smallest and largest numbers
        s = rng.choice(np.array([0.0, -0.0, np.inf, -np.inf, np.nan, 1e-45, -1e-45, 3.4e38, -3.4e38, 1.0, 1.0000001]), n)
    rng.shuffle(s)
    return s.astype(np.float32)


@pytest.mark.parametrize("kind", ["dense", "crowd", "tied crowd", "edge", "outliers", "top", "odd"])
@pytest.mark.parametrize("n", [1, 2, 64, 1025, 4096, 4097, 8192, 8193, 16384])
def test_every_end(n, kind):
    rng = np.random.default_rng(n)
    s = _scores(kind, n, rng)
    rank = int((s > 3.0).sum()) if kind not in ("odd", "outliers", "top") else n // 2
    cuts = sorted({min(n, max(0, k)) for k in (0, 1, n // 3, n - 1, n, rank, rank - 1, rank - 64, rank - 65, rank - 499, rank - 500, rank - 501)})
    if kind == "edge":             # inside either block, from both ends
        cuts = sorted({*cuts, *(k for i in (1, 17, 32, 63, 64, 65, 66, 97, 128, 129) for k in (i + 1, n - 1 - i) if 0 <= k <= n)})
    dev = torch.from_numpy(s).cuda()
    halt, counts = torch.empty((n,), dtype=torch.uint8, device="cuda"), torch.empty(((n + 63) // 64,), dtype=torch.int32, device="cuda")
    ws = torch.empty((256 + 4 * counts.numel(),), dtype=torch.uint8, device="cuda")
    for k in cuts:
        for prot in ((0, 0), (min(n, 3), min(n, 2))):
            p = B.make_params(512, 4, 4, 128, rule=B.RULE_TOPK, k_keep=k, keep_first_n=prot[0], keep_last_n=prot[1])
            for low in (False, True):
                B.dash_decide_topk(p, dev, n, low, halt, counts, ws)
                want = np.asarray(ref.decide_topk(s, k, prot[0], prot[1], keep_low=low)).astype(np.uint8)
                assert np.array_equal(halt.cpu().numpy(), want), (n, kind, k, prot, low)
                kept = np.add.reduceat((want == 0).astype(np.int32), np.arange(0, n, 64))
                assert np.array_equal(counts.cpu().numpy(), kept)
