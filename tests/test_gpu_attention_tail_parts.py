"""Layer calls without a causal mask whose last rows take the few-row form, their keys cut over several workgroups or not, against fp64: the
projection is the identity and x zero, so x_next holds the attention's result."""
import pytest

torch = pytest.importorskip("torch")
from paper_2604_18103_amd import binding as B
from test_attention_form import ONE_AND_TAIL
from test_attention_tail_parts import layer_scratch, parts_of
from test_staging_addresses import _load

pytestmark = pytest.mark.gpu


# rows, query and key/value heads, head size, parts of the last rows' keys (more than half of the units in workgroups: not cut)
@pytest.mark.parametrize("n,hq,hkv,dh,parts", [(4097, 16, 4, 64, 9), (4129, 16, 4, 64, 6), (8200, 16, 4, 64, 11), (4319, 16, 4, 64, 2),
                                               (2785, 24, 8, 64, 1), (2305, 28, 4, 128, 5), (2337, 28, 4, 128, 4), (4609, 28, 4, 128, 7),
                                               (2433, 28, 4, 128, 1)])
@pytest.mark.parametrize("infinite", [None, slice(0, 1024), slice(2048, 5000)])
def test_last_rows(n, hq, hkv, dh, parts, infinite):
    """P and the result are rounded to bf16, 2.3e-3 of a row (test_gpu_attention_few): 3e-3 on the mean, 8e-3 on the largest. Keys without
    a finite score fill whole parts, the first ones and the last ones."""
    cu, d = torch.cuda.get_device_properties(0).multi_processor_count, hq * dh
    p = B.make_params(d, hq, hkv, dh, causal=False, rule=B.RULE_NONE)
    buf = B.alloc_layer_buffers(p, n)
    assert _load().dash_fa_form(n, hq, dh, 0, cu) == ONE_AND_TAIL and _load().dash_fa_few_tail(n, hq, dh, cu)
    g = torch.Generator(device="cuda").manual_seed(n)
    q, k, v = (torch.randn((n, h, dh), generator=g, device="cuda").bfloat16() for h in (hq, hkv, hkv))
    if infinite is not None:
        q[:, :, 0], k[:, :, 0] = 1.0, 0.0
        k[infinite, :, 0] = float("-inf")
    assert parts_of(n, hq, dh, cu, layer_scratch(n, d, d))[0] == parts
    x, idx = torch.zeros((n, d), dtype=torch.bfloat16, device="cuda"), torch.arange(n, dtype=torch.int32, device="cuda")
    B.dash_attn_layer(p, x, q, k, v, torch.eye(d, dtype=torch.bfloat16, device="cuda"), idx, n, buf)
    r0 = n - n % 256
    got = buf.x_next[r0:n].double().reshape(-1, hq, dh)
    want = torch.empty_like(got)
    for h in range(hq):
        kh, vh = k[:, h // (hq // hkv)].double(), v[:, h // (hq // hkv)].double()
        s = q[r0:, h].double() @ kh.t().contiguous() * dh ** -0.5
        want[:, h] = torch.softmax(s, dim=1) @ vh
    err = (got - want).norm(dim=2) / want.norm(dim=2)
    assert float(err.max()) <= 8e-3 and float(err.mean()) <= 3e-3


@pytest.mark.parametrize("n,hq,hkv,dh", [(4097, 16, 4, 64), (2305, 28, 4, 128)])
def test_with_the_debug_output_the_stage_calls_bits(n, hq, hkv, dh):
    """With delta_dbg the layer call adds in the order of the stage-level calls, attention included."""
    d, bf = hq * dh, torch.bfloat16
    p = B.make_params(d, hq, hkv, dh, causal=False, rule=B.RULE_NONE)
    g = torch.Generator(device="cuda").manual_seed(n)
    rnd = lambda *shape: torch.randn(shape, generator=g, device="cuda").to(bf)
    q, k, v, x, w = rnd(n, hq, dh), rnd(n, hkv, dh), rnd(n, hkv, dh), rnd(n, d), rnd(d, d)
    idx = torch.arange(n, dtype=torch.int32, device="cuda")
    buf = B.alloc_layer_buffers(p, n, with_delta=True)
    B.dash_attn_layer(p, x, q, k, v, w, idx, n, buf)
    o, x_next, delta = (torch.empty((n, d), dtype=t, device="cuda") for t in (bf, bf, torch.float32))
    partials = torch.empty((B.norm_partials_per_row(p), n, 2), dtype=torch.float32, device="cuda")
    B.dash_flash_fwd(p, q, k, v, idx, n, o)
    B.dash_wo_residual_rownorm(p, o, w, x, n, x_next, partials, delta)
    assert torch.equal(buf.x_next[:n], x_next) and torch.equal(buf.delta_dbg[:n], delta)
