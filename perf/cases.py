"""The work whose speed counts: what a program that prefills with halting has this library do, through its public
entry points, over the range of lengths, shapes, types and options that it meets.

Four paths:
  layer     binding.dash_attn_layer: attention, projection + residual, score, decision, compaction of one layer
  chain     chain.run_chain: one layer of the attention-only chain, with its front end (RMSNorm, q/k/v, rotary
            embedding) and the read-back of the survivor count
  schedule  single_shot.run_schedule (or its captured graph): whole blocks with a halting decision after some
  signal    the ablation's route: block-level score of stored rows, TopK on given scores, compaction, and the halted
            rows scattered to their original positions

Sizes are those of the repository's configurations, tests and benchmark. Values are the benchmark's distributions
(heavy-tailed row norms, normal q / k / v and weights), drawn on the device from the seed.

Which rows halt is a comparison of scores, so two correct implementations may disagree on a row whose score lies
within rounding of the cut, and everything after that row in the compacted output would then sit one place further.
The cut of every case is therefore put into the widest gap between neighbouring scores near the wanted fraction; the
scores for that come from plain torch operations in 32-bit arithmetic, not from the library.
"""
from __future__ import annotations

import math

import torch

from paper_2604_18103_amd import binding as B
from paper_2604_18103_amd import chain as CH
from paper_2604_18103_amd import single_shot as SS

# hidden size, query heads, key/value heads, head size, feed-forward width (0: the shape is not used in whole blocks)
SHAPES = {
    "tiny": (256, 4, 1, 64, 0),          # the fp32 configuration
    "small": (512, 4, 2, 128, 1408),     # the smoke test's layer; the tests' feed-forward
    "narrow": (1024, 16, 4, 64, 0),      # head size 64
    "qwen": (3584, 28, 4, 128, 18944),   # Qwen2.5-7B
    "llama": (4096, 32, 8, 128, 0),      # Llama-3-8B
}
THETA = 1.0e6


def _layer(name, shape, n, prompt, dtype="bf16", causal=True, rule="threshold", score="rel", halt=0.5, first=0, last=0):
    return dict(name=name, path="layer", shape=shape, n=n, prompt=prompt, dtype=dtype, causal=causal, rule=rule,
                score=score, halt=halt, first=first, last=last)


def listed():
    return [
        # the fp32 configuration: a short prompt in full precision
        _layer("layer_tiny_f32", "tiny", 512, 512, dtype="f32"),
        # a short prompt in bf16, odd length: launches and latency
        _layer("layer_small_333", "small", 333, 1024, halt=0.4),
        # what is left of an 8k prompt after 99 % halted, decided by rank with the protected ends
        _layer("layer_qwen_177", "qwen", 177, 8192, rule="topk", halt=0.3, first=64, last=32),
        # ... and after 75 % halted
        _layer("layer_qwen_2120", "qwen", 2120, 8192, rule="topk", halt=0.3, first=64, last=32),
        # an 8k prompt before anything halted
        _layer("layer_qwen_8k", "qwen", 8192, 8192, halt=0.6),
        # the headline: a 32k prompt, half of it still active
        _layer("layer_qwen_32k_half", "qwen", 16384, 32768, halt=0.3),
        # the longest context, 40 % active
        _layer("layer_llama_128k_40", "llama", 52428, 131072, halt=0.5),
        # bidirectional attention, head size 64, absolute scores, nothing halts (layers before the start layer)
        _layer("layer_narrow_full", "narrow", 4097, 4097, causal=False, rule="none", score="abs"),
        # the last layer of the eight-layer chain on a 32k prompt
        dict(name="chain_qwen_6874", path="chain", shape="qwen", n=6874, prompt=32768, halt=0.2),
        # an 8k prompt at an extreme ratio (88.89 % halted): one full block, then short ones, replayed from a graph
        dict(name="schedule_qwen_8k_graph", path="schedule", shape="qwen", n=8192, blocks=3, shots=1, keep=0.1111,
             first=64, last=32, graph=True),
        # the single-shot setting: a full block of a 32k prompt with the decision, and a block on what is kept
        dict(name="schedule_qwen_32k", path="schedule", shape="qwen", n=32768, blocks=2, shots=1, keep=0.335,
             first=64, last=32, graph=False),
        # the block-level signal on the headline's rows
        dict(name="signal_qwen_16k", path="signal", shape="qwen", n=16384, prompt=32768, halt=0.3, keep_low=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: the same paths, lengths over their range on a logarithmic scale (odd as well as even), shapes
    and options as they come up together."""
    path = rng.choice(["layer"] * 6 + ["chain"] * 2 + ["schedule"] * 2 + ["signal"])
    if path == "layer":
        shape = rng.choice(["tiny", "small", "narrow", "qwen", "qwen", "qwen", "llama"])
        dtype = "f32" if shape == "tiny" or (shape == "small" and rng.random() < 0.3) else "bf16"
        n = _log_int(rng, 16, {"tiny": 2048, "small": 2048, "narrow": 8192}.get(shape, 32768))
        guard = n > 200 and rng.random() < 0.4
        return dict(path=path, shape=shape, n=n, prompt=int(n * rng.uniform(1.0, 3.0)), dtype=dtype,
                    causal=rng.random() < 0.85, rule=rng.choice(["threshold", "topk", "none"]),
                    score=rng.choice(["rel", "rel", "abs"]), halt=round(rng.uniform(0.1, 0.8), 3),
                    first=64 if guard else 0, last=32 if guard else 0)
    if path == "chain":
        shape = rng.choice(["small", "qwen", "qwen"])
        n = _log_int(rng, 64, 16384)
        return dict(path=path, shape=shape, n=n, prompt=int(n * rng.uniform(1.0, 3.0)), halt=round(rng.uniform(0.1, 0.5), 3))
    if path == "schedule":
        shape = rng.choice(["small", "qwen", "qwen"])
        blocks = rng.randint(2, 3)
        return dict(path=path, shape=shape, n=_log_int(rng, 512, 12288), blocks=blocks, shots=rng.randint(1, blocks - 1),
                    keep=round(math.exp(rng.uniform(math.log(0.03), math.log(0.6))), 4),
                    first=64, last=32, graph=rng.random() < 0.5)
    n = _log_int(rng, 512, 65536)
    return dict(path=path, shape=rng.choice(["small", "qwen", "llama"]), n=n, prompt=int(n * rng.uniform(1.0, 3.0)),
                halt=round(rng.uniform(0.1, 0.8), 3), keep_low=rng.random() < 0.25)


# ---------------------------------------------------------------- inputs

def _hidden(g, n, d, dtype, mixed=False):
    """Rows g_t exp(mu + sigma z_t): heavy-tailed norms; `mixed`: 80 % of the rows around a larger norm."""
    z = torch.randn((n, 1), generator=g, device="cuda")
    f = 1.5 * z
    if mixed:
        f = torch.where(torch.rand((n, 1), generator=g, device="cuda") < 0.8, 1.0 + 0.5 * z, f)
    return (torch.randn((n, d), generator=g, device="cuda") * torch.exp(f)).to(dtype)


def _normal(g, shape, dtype, fan=1):
    return (torch.randn(shape, generator=g, device="cuda") * fan ** -0.5).to(dtype)


def _positions(g, prompt, n):
    return torch.sort(torch.randperm(prompt, generator=g, device="cuda")[:n]).values.to(torch.int32)


# ---------------------------------------------------------------- scores in plain torch, to place the cut

def _attention(q, k, v, causal, dt=torch.float32):
    n, hq, dh = q.shape
    group = hq // k.shape[1]
    q, k, v = q.to(dt), k.to(dt), v.to(dt)
    out = torch.empty_like(q)
    rank = torch.arange(n, device=q.device)
    for h in range(hq):
        kt, vh = k[:, h // group].contiguous().t(), v[:, h // group].contiguous()
        for r0 in range(0, n, 2048):
            r1 = min(n, r0 + 2048)
            end = r1 if causal else n
            s = (q[r0:r1, h] * dh ** -0.5) @ kt[:, :end]
            if causal:
                s[:, r0:].masked_fill_(rank[r0:end] > rank[r0:r1, None], float("-inf"))
            out[r0:r1, h] = torch.softmax(s, dim=1) @ vh[:end]
    return out.reshape(n, hq * dh)


def _scores(delta, x, kind):
    s = delta.norm(dim=1)
    return s / x.to(s.dtype).norm(dim=1) if kind == "rel" else s


def _rms(x, dt=torch.float32):
    x = x.to(dt)
    return x * torch.rsqrt((x * x).mean(dim=1, keepdim=True) + 1e-6)


def _rope(u, pos):
    half = u.shape[2] // 2
    freq = THETA ** (-torch.arange(half, device=u.device, dtype=torch.float64) / half)
    a = pos.double()[:, None] * freq
    c, s = torch.cos(a).to(u.dtype)[:, None], torch.sin(a).to(u.dtype)[:, None]
    lo, hi = u[..., :half], u[..., half:]
    return torch.cat([lo * c - hi * s, lo * s + hi * c], dim=2)


def _front(x, w_qkv, pos, hq, hkv, dh, dt=torch.float32):
    u = _rms(x, dt) @ w_qkv.to(dt)
    q, k, v = (t.reshape(x.shape[0], -1, dh) for t in u.split([hq * dh, hkv * dh, hkv * dh], dim=1))
    return _rope(q, pos), _rope(k, pos), v


def _ffn(x, gate, up, down, dt=torch.float32):
    out = []
    gate, up, down = gate.to(dt), up.to(dt), down.to(dt)
    for r in x.split(4096):
        h = _rms(r, dt)
        out.append(r + (torch.nn.functional.silu(h @ gate) * (h @ up)) @ down)
    return torch.cat(out)


def _cut(scores, halt, first=0, last=0):
    """(threshold, rows kept): the widest relative gap between neighbouring scores of the unprotected rows within a
    twentieth of the wanted halted fraction."""
    n = scores.numel()
    s = torch.sort(scores[first:n - last].double()).values.cpu()
    m = s.numel()
    at, reach = int(halt * m), max(1, m // 20)
    lo, hi = max(1, at - reach), min(m - 1, at + reach)
    if m < 2 or lo > hi:
        return 0.0, n
    i = lo + int(torch.argmax(torch.log(s[lo:hi + 1] / s[lo - 1:hi])))
    return float(torch.sqrt(s[i - 1] * s[i])), n - i


# ---------------------------------------------------------------- preparation

def _outputs(buf):
    """The buffers a layer call fills. Only the survivors' part of the compacted ones is written: the rest is zero."""
    buf.x_compact.zero_()
    buf.new_active_idx.zero_()
    return [buf.x_next, buf.scores, buf.halt_mask, buf.x_compact, buf.new_active_idx, buf.n_active_out]


def _prepare_layer(case, g):
    d, hq, hkv, dh, _ = SHAPES[case["shape"]]
    n = case["n"]
    lib_dtype = B.DASH_F32 if case["dtype"] == "f32" else B.DASH_BF16
    dt = B.torch_dtype(lib_dtype)
    x = _hidden(g, n, d, dt, mixed=case["shape"] == "llama")
    q, k, v = (_normal(g, (n, h, dh), dt) for h in (hq, hkv, hkv))
    w_o = _normal(g, (hq * dh, d), dt, d)
    idx = _positions(g, case["prompt"], n)
    tau, kept = 0.0, n
    if case["rule"] != "none":
        delta = _attention(q, k, v, case["causal"]) @ w_o.float()
        tau, kept = _cut(_scores(delta, x, case["score"]), case["halt"], case["first"], case["last"])
    rule = {"none": B.RULE_NONE, "threshold": B.RULE_THRESHOLD, "topk": B.RULE_TOPK}[case["rule"]]
    p = B.make_params(d, hq, hkv, dh, dtype=lib_dtype, causal=case["causal"], rule=rule,
                      score_kind=B.SCORE_REL if case["score"] == "rel" else B.SCORE_ABS, tau=tau, k_keep=kept,
                      keep_first_n=case["first"], keep_last_n=case["last"])
    buf = B.alloc_layer_buffers(p, n)
    return dict(args=(p, x, q, k, v, w_o, idx, n, buf), out=_outputs(buf))


def _prepare_chain(case, g):
    d, hq, hkv, dh, _ = SHAPES[case["shape"]]
    n, bf = case["n"], torch.bfloat16
    x = _hidden(g, n, d, bf)
    idx = _positions(g, case["prompt"], n)
    w = dict(w_qkv=_normal(g, (d, (hq + 2 * hkv) * dh), bf, d), w_o=_normal(g, (hq * dh, d), bf, d))
    delta = _attention(*_front(x, w["w_qkv"], idx, hq, hkv, dh), True) @ w["w_o"].float()
    _, kept = _cut(_scores(delta, x, "rel"), case["halt"])
    state = CH.alloc_chain(d, hq, hkv, dh, n)
    return dict(args=(state, x, idx, n, [w], (n - kept + 0.5) / n), out=_outputs(state.bufs[0]))


def _prepare_schedule(case, g):
    d, hq, hkv, dh, m = SHAPES[case["shape"]]
    n, bf = case["n"], torch.bfloat16
    x0 = _hidden(g, n, d, bf)
    x, pos = x0.float(), torch.arange(n, device="cuda")
    weights, shots = [], {}
    for l in range(case["blocks"]):
        w = dict(w_qkv=_normal(g, (d, (hq + 2 * hkv) * dh), bf, d), w_o=_normal(g, (hq * dh, d), bf, d))
        gate, up = _normal(g, (d, m), bf, d), _normal(g, (d, m), bf, d)
        w["w_down"] = _normal(g, (m, d), bf, m)
        w["w_gate_up"] = B.interleave_gate_up(gate, up)
        weights.append(w)
        if l < case["shots"]:  # decisions after the first blocks: the rows of each have to be known to place its cut
            delta = _attention(*_front(x, w["w_qkv"], pos, hq, hkv, dh), True) @ w["w_o"].float()
            scores = _scores(delta, x, "rel")
            kept = x.shape[0]  # a few hundred rows are not cut again
            if kept > 400:
                _, kept = _cut(scores, 1.0 - case["keep"], case["first"], case["last"])
            shots[l] = kept
            if l + 1 < case["shots"]:
                inner = scores.clone()
                inner[:case["first"]] = inner[inner.numel() - case["last"]:] = float("inf")
                keep = torch.sort(torch.topk(inner, kept).indices).values
                x, pos = _ffn((x + delta)[keep], gate, up, w["w_down"]), pos[keep]
        del gate, up
    st = SS.alloc_blocks(d, hq, hkv, dh, m, n)
    st.params.keep_first_n, st.params.keep_last_n = case["first"], case["last"]
    final = torch.zeros_like(x0)
    if case["graph"]:
        prompt = x0.clone()
        return dict(graph=SS.GraphedSchedule(st, x0, weights, shots, rope_theta=THETA, final=final), x0=x0,
                    prompt=prompt, final=final, weights=weights, shots=shots)
    return dict(args=(st, x0, weights, shots, THETA, final), final=final)


def _prepare_signal(case, g):
    d, hq, hkv, dh, _ = SHAPES[case["shape"]]
    n, bf = case["n"], torch.bfloat16
    old = _hidden(g, n, d, bf)
    new = (old.float() + _normal(g, (n, d), torch.float32) * 0.3).to(bf)
    idx = _positions(g, case["prompt"], n)
    diff, low = _scores(new.float() - old.float(), old, "rel"), case["keep_low"]
    _, kept = _cut(1.0 / diff if low else diff, case["halt"])
    p = B.make_params(d, hq, hkv, dh, rule=B.RULE_TOPK, k_keep=kept)
    chunks = (n + B.CHUNK_ROWS - 1) // B.CHUNK_ROWS
    s = dict(p=p, old=old, new=new, idx=idx, n=n, d=d, low=low, prompt=case["prompt"],
             scores=torch.empty((n,), dtype=torch.float32, device="cuda"),
             halt=torch.empty((n,), dtype=torch.uint8, device="cuda"),
             counts=torch.empty((chunks,), dtype=torch.int32, device="cuda"),
             ws=torch.empty((256 + 4 * chunks,), dtype=torch.uint8, device="cuda"),
             compact=torch.zeros((n, d), dtype=bf, device="cuda"),
             new_idx=torch.zeros((n,), dtype=torch.int32, device="cuda"),
             n_out=torch.zeros((1,), dtype=torch.int32, device="cuda"),
             full=torch.zeros((case["prompt"], d), dtype=bf, device="cuda"))
    s["out"] = [s["scores"], s["halt"], s["compact"], s["new_idx"], s["n_out"], s["full"]]
    return s


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    make = dict(layer=_prepare_layer, chain=_prepare_chain, schedule=_prepare_schedule, signal=_prepare_signal)
    return dict(make[case["path"]](case, g), path=case["path"])


# ---------------------------------------------------------------- one pass

def run(state):
    path = state["path"]
    if path == "layer":
        B.dash_attn_layer(*state["args"])
        return state["out"]
    if path == "chain":
        chain, x, idx, n, weights, halt = state["args"]
        CH.run_chain(chain, x, idx, n, weights, halt, rope_theta=THETA)
        return state["out"]
    if path == "schedule":
        if "graph" in state:
            state["x0"].copy_(state["prompt"])
            state["graph"].replay()
            return [state["final"]]
        st, x0, weights, shots, theta, final = state["args"]
        res = SS.run_schedule(st, x0, weights, shots, rope_theta=theta, final=final)
        return [final, res["n_after"]]
    s = state
    B.dash_score_diff_rows(s["new"], s["old"], s["n"], s["d"], B.DASH_BF16, B.SCORE_REL, s["scores"])
    B.dash_decide_topk(s["p"], s["scores"], s["n"], s["low"], s["halt"], s["counts"], s["ws"])
    B.dash_compact(s["p"], s["halt"], s["counts"], s["idx"], s["new"], s["n"], s["compact"], s["new_idx"], s["n_out"])
    B.dash_scatter_rows(s["new"], s["idx"], s["halt"], 1, s["n"], s["d"], B.DASH_BF16, s["prompt"], s["full"])
    return s["out"]


# ---------------------------------------------------------------- what a pass cannot do without

def work(case):
    d, hq, hkv, dh, m = SHAPES[case["shape"]]
    n, da, dkv = case["n"], hq * dh, hkv * dh

    def attention(rows, causal=True):
        return 4.0 * da * (rows * (rows + 1) / 2 if causal else rows * rows)

    if case["path"] == "layer":
        e = 4 if case["dtype"] == "f32" else 2
        kept = n if case["rule"] == "none" else n - case["halt"] * (n - case["first"] - case["last"])
        return dict(flops=attention(n, case["causal"]) + 2.0 * n * da * d,
                    bytes=e * (n * (2 * d + da + 2 * dkv) + da * d + kept * d) + n * (4 + 4 + 1) + 4 * kept)
    if case["path"] == "chain":
        kept = n - case["halt"] * n
        return dict(flops=attention(n) + 2.0 * n * d * (2 * da + 2 * dkv),
                    bytes=2 * (2 * n * d + kept * d + d * (2 * da + 2 * dkv)) + n * (4 + 4 + 1) + 4 * kept)
    if case["path"] == "schedule":
        flops, rows = 0.0, n
        for l in range(case["blocks"]):
            flops += attention(rows) + 2.0 * rows * d * (2 * da + 2 * dkv) + 6.0 * rows * d * m
            if l < case["shots"] and rows > 400:
                guard = case["first"] + case["last"]
                rows = guard + case["keep"] * (rows - guard)
        return dict(flops=flops, bytes=2 * (2 * n * d + case["blocks"] * (d * (2 * da + 2 * dkv) + 3 * d * m)))
    kept = n - case["halt"] * n
    return dict(flops=3.0 * n * d, bytes=2 * (2 * n * d + n * d) + n * (4 + 4 + 1) + 4 * kept)


def tolerance(case):
    """About four times what the paths measure against the plain torch computation of the same step in 32 bits:
    rows up to 1e-3 (one bf16 rounding each, at most one step, 2^-7, of an element), scores up to 1e-3; whole blocks,
    whose rows are rounded several times, 2.5e-3 and 2e-2 of an element; 32-bit paths 1.2e-7 and 1.2e-6, for sums in
    another order. Flags, counts and positions are the same: no cut lies near a score."""
    if case["path"] == "signal" or (case["path"] == "layer" and case["dtype"] == "f32"):
        return dict(rel=1e-6, max=1e-5)
    if case["path"] == "schedule":
        return dict(rel=1e-2, max=8e-2)
    return dict(rel=4e-3, max=3e-2)


# ---------------------------------------------------------------- the same pass in 64 bits, in plain torch

def _kept(scores, k_keep, first, last, low=False):
    """TopK: the protected rows and the best of the others, k_keep in all, in their order."""
    s = -scores if low else scores.clone()
    s[:first] = float("inf")
    s[s.numel() - last:] = float("inf")
    return torch.sort(torch.topk(s, max(k_keep, min(first + last, s.numel()))).indices).values


def _decided(scores, kept, idx, rows):
    """The outputs that follow from which rows are kept: flags, compacted rows and positions, count."""
    halt = torch.ones(scores.shape, dtype=torch.uint8, device="cuda")
    halt[kept] = 0
    compact, new_idx = torch.zeros_like(rows), torch.zeros_like(idx)
    compact[:kept.numel()], new_idx[:kept.numel()] = rows[kept], idx[kept]
    return [halt, compact, new_idx, torch.full((1,), kept.numel(), dtype=torch.int32, device="cuda")]


def exact(case, seed):
    f64 = torch.float64
    d, hq, hkv, dh, m = SHAPES[case["shape"]]
    state = prepare(case, seed)
    if case["path"] == "layer":
        p, x, q, k, v, w_o, idx, n, _ = state["args"]
        delta = _attention(q, k, v, case["causal"], f64) @ w_o.to(f64)
        scores, first, last = _scores(delta, x, case["score"]), case["first"], case["last"]
        if case["rule"] == "topk":
            kept = _kept(scores, int(p.k_keep), first, last)
        else:
            stays = scores >= (float(p.tau) if case["rule"] == "threshold" else 0.0)
            stays[:first] = stays[n - last:] = True
            kept = torch.nonzero(stays)[:, 0]
        x_next = x.to(f64) + delta
        return [x_next, scores] + _decided(scores, kept, idx, x_next)
    if case["path"] == "chain":
        _, x, idx, n, weights, halt = state["args"]
        delta = _attention(*_front(x, weights[0]["w_qkv"], idx, hq, hkv, dh, f64), True, f64) @ weights[0]["w_o"].to(f64)
        scores, x_next = _scores(delta, x, "rel"), x.to(f64) + delta
        return [x_next, scores] + _decided(scores, _kept(scores, n - int(halt * n), 0, 0), idx, x_next)
    if case["path"] == "schedule":
        if case["graph"]:
            x0, weights, shots = state["prompt"], state["weights"], state["shots"]
        else:
            _, x0, weights, shots, _, _ = state["args"]
        x, pos = x0.to(f64), torch.arange(x0.shape[0], device="cuda")
        final = torch.empty_like(x)
        for l, w in enumerate(weights):
            gate, up = (t.reshape(d, m) for t in w["w_gate_up"].reshape(d, m // 32, 2, 32).unbind(2))
            delta = _attention(*_front(x, w["w_qkv"], pos, hq, hkv, dh, f64), True, f64) @ w["w_o"].to(f64)
            done = _ffn(x + delta, gate, up, w["w_down"], f64)
            if l in shots:
                final[pos] = done
                kept = _kept(_scores(delta, x, "rel"), shots[l], case["first"], case["last"])
                done, pos = done[kept], pos[kept]
            x = done
        final[pos] = x
        return [final] if case["graph"] else [final, x.shape[0]]
    old, new, idx, low = state["old"], state["new"], state["idx"], state["low"]
    scores = _scores(new.to(f64) - old.to(f64), old, "rel")
    kept = _kept(scores, int(state["p"].k_keep), 0, 0, low)
    out = _decided(scores, kept, idx, new.to(f64))
    full = torch.zeros(state["full"].shape, dtype=f64, device="cuda")
    gone = out[0] == 1
    full[idx[gone].long()] = new[gone].to(f64)
    return [scores] + out + [full]
