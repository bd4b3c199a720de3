"""The layer call's TOPK rule where scores, decision and compaction are one launch (up to 4096 rows, at lengths of chunks and a few hundred
rows; longer ones: test_gpu_topk_compact.py): against the oracle's TopK on the GPU's own scores, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import reference as ref
from paper_2604_18103_amd import binding as B

pytestmark = pytest.mark.gpu


def _layer(n, d, hq, k_keep, prot, kind, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    bf = torch.bfloat16
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    x = (rnd(n, d) * torch.exp(1.5 * rnd(n, 1))).to(bf)
    q, k, v = (rnd(n, hq, 64).to(bf) for _ in range(3))
    w_o = (rnd(hq * 64, d) / d ** 0.5).to(bf)
    if kind == "tied":            # every row the same score
        w_o.zero_()
    elif kind == "nan":           # every row from the middle on sees a NaN value: NaN scores rank highest and tie
        v[n // 2] = float("nan")
    elif kind == "few":           # a handful of different rows: ties in groups
        x = x[torch.arange(n, device="cuda") % 5].contiguous()
        v[:] = v[0]
    idx = torch.arange(0, 3 * n, 3, dtype=torch.int32, device="cuda")
    p = B.make_params(d, hq, hq, 64, rule=B.RULE_TOPK, k_keep=k_keep, keep_first_n=prot[0], keep_last_n=prot[1])
    buf = B.alloc_layer_buffers(p, n)
    for _ in range(2):            # twice on the same workspace: the words of the first call are cleared by the second
        B.dash_attn_layer(p, x, q, k, v, w_o, idx, n, buf)
    torch.cuda.synchronize()
    scores = buf.scores[:n].cpu().numpy()
    want = np.asarray(ref.decide_topk(scores, k_keep, prot[0], prot[1])).astype(np.uint8)
    assert np.array_equal(buf.halt_mask[:n].cpu().numpy(), want), (n, k_keep, prot, kind)
    kept = np.flatnonzero(want == 0)
    assert int(buf.n_active_out.item()) == kept.size
    kt = torch.from_numpy(kept).cuda()
    assert torch.equal(buf.new_active_idx[:kept.size], idx[kt])
    got, rows = buf.x_compact[:kept.size], buf.x_next[kt]
    assert torch.equal(got.view(torch.int16), rows.view(torch.int16))
    # the stage-level decision on the same scores
    counts = torch.empty(((n + 63) // 64,), dtype=torch.int32, device="cuda")
    halt = torch.empty((n,), dtype=torch.uint8, device="cuda")
    ws = torch.empty((256 + 4 * counts.numel(),), dtype=torch.uint8, device="cuda")
    B.dash_decide_topk(p, buf.scores[:n].contiguous(), n, False, halt, counts, ws)
    assert torch.equal(halt, buf.halt_mask[:n])


@pytest.mark.parametrize("n", [1, 63, 64, 65, 255, 257, 513, 704, 705, 767, 768, 769, 1000, 1472, 1473, 1535, 1536, 1537])
def test_against_the_oracle(n):
    for i, (k_keep, prot) in enumerate(((n // 3, (0, 0)), (n, (0, 0)), (0, (0, 0)), (max(1, n // 2), (min(n, 5), min(n, 3))),
                                        (2, (min(n, 64), min(n, 32))))):
        _layer(n, 64 if n > 1500 or n == 768 else 264, 1, k_keep, prot, "spread", seed=n + i)


@pytest.mark.parametrize("kind", ["tied", "nan", "few"])
def test_ties_and_nans(kind):
    for n, k_keep, prot in ((200, 77, (0, 0)), (333, 150, (10, 7)), (700, 650, (64, 32)), (1500, 1400, (64, 32)), (130, 1, (0, 0))):
        _layer(n, 128, 2, k_keep, prot, kind, seed=n)
