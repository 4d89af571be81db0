"""Performance cases of the MoE layer: what is timed, through the library's public entry points.

Three kinds of call:
  layer  one zeda_moe_forward (route, dispatch, expert FFN, combine), weights kept as a serving program keeps them
  stack  MoeStack.forward: layers chained as x <- x + MoE(RMSNorm(x)), the block form of the layer
  stats  zeda_routing_stats: the batch statistics that a load-balance monitor reads

A case is a dict of plain values.  Layer shapes are the ones the package's own configurations and tests use
(synth.CONFIGS): H=2048, I=768, N=128, K=8 with 32 or 64 zero experts; H=2048, I=1536, N=64, K=4 with 32; and small
layers whose widths are not multiples of the large tiles.  About half of the slots land on zero experts.
"""
from __future__ import annotations

import math

import torch

from paper_2605_18643_amd import synth, zeda
from paper_2605_18643_amd.stack import EPS, MoeStack

GATES = {"softmax": zeda.GATE_SOFTMAX, "topk_norm": zeda.GATE_TOPK_NORM, "real_renorm": zeda.GATE_REAL_RENORM}
# bias on every zero expert's logit that puts half of the slots on zero experts when the logits have a standard
# deviation of 0.905 (router weights of 0.02 at H = 2048; other widths scale the weights to keep it)
ZERO_BIAS = {(128, 32, 8): synth.QWEN_ZERO_BIAS, (128, 64, 8): synth.NZ64_ZERO_BIAS, (64, 32, 4): synth.GLM_LIKE_ZERO_BIAS}
LOGIT_STD = 0.02 * math.sqrt(2048.0)
MIN_GAP = 2e-4  # between a token's K-th and next logit: fp32 sums in any order then select the same set

WIDE = dict(H=2048, I=768, N=128, Z=32, K=8)
WIDE64 = dict(H=2048, I=768, N=128, Z=64, K=8)
FEW = dict(H=2048, I=1536, N=64, Z=32, K=4)


def _layer(name, T, shape, dtype="bf16", layout="tiled", gate="topk_norm", copy=False, recipe="zero_bias"):
    c = dict(kind="layer", T=T, dtype=dtype, layout=layout, gate=gate, copy=copy, recipe=recipe, **shape)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the fp32 reference layer of the tests: a handful of rows per expert, nothing but latency
        _layer("f32_tiny_64", 64, dict(H=256, I=128, N=8, Z=4, K=2), dtype="f32", layout="row_major", recipe="plain"),
        # an fp32 layer of working size (checking a converted checkpoint in full precision), ragged token count
        _layer("f32_layer_513", 513, dict(H=1024, I=512, N=32, Z=8, K=4), dtype="f32", layout="row_major"),
        # decode of one sequence: the smallest serving call
        _layer("decode_1", 1, WIDE),
        # decode at concurrency 32, the paper's N_Z = 64, weights as they come out of a checkpoint (not packed)
        _layer("decode_32_rowmajor", 32, WIDE64, layout="row_major"),
        # decode at concurrency 64: streams nearly every expert's weights
        _layer("decode_64", 64, WIDE),
        # small model with widths that only the narrow tiles divide, copy experts (Appendix B) and Eq. 7's weights
        _layer("ragged_301_copy", 301, dict(H=1152, I=448, N=24, Z=8, K=3), layout="row_major", gate="real_renorm", copy=True),
        # a prefill chunk of odd length (chunked prefill beside decodes): about 31 rows per expert
        _layer("prefill_997", 997, WIDE),
        # the benchmark layer: prefill of 4096 tokens
        _layer("prefill_4096", 4096, WIDE),
        # the router of the paper's second model, weights not packed, gates as plain softmax
        _layer("prefill_4096_few_rowmajor", 4096, FEW, layout="row_major", gate="softmax"),
        # heterogeneous difficulty and Zipf(1.1) expert popularity: 16384 tokens, loads from tens to thousands of rows
        _layer("hetero_16384", 16384, WIDE, recipe="planted"),
        # four chained layers at 8192 tokens (residual and norm folded into the combine)
        dict(name="stack_4x8192", kind="stack", T=8192, layers=4, dtype="bf16", layout="tiled", **WIDE),
        # routing statistics of a batch of 8192 tokens (load-balance monitoring)
        dict(name="stats_8192", kind="stats", T=8192, dtype="bf16", **WIDE),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "layer", "f32", "small", "stack", "stats"])
    if kind == "f32":
        shape = dict(H=4 * rng.randint(64, 256), I=4 * rng.randint(32, 128), N=rng.randint(8, 32), Z=rng.randint(0, 8), K=rng.randint(1, 4))
        return _layer(None, _log_int(rng, 1, 256), shape, dtype="f32", layout="row_major", gate=rng.choice(sorted(GATES)),
                      copy=rng.random() < 0.3, recipe="plain")
    if kind == "small":
        shape = dict(H=128 * rng.randint(2, 12), I=64 * rng.randint(2, 12), N=rng.randint(8, 48), Z=rng.randint(0, 16), K=rng.randint(1, 6))
        return _layer(None, _log_int(rng, 1, 4096), shape, layout=rng.choice(["tiled", "row_major"]), gate=rng.choice(sorted(GATES)),
                      copy=rng.random() < 0.3, recipe="plain")
    if kind == "stack":
        return dict(kind="stack", T=_log_int(rng, 1, 6144), layers=rng.randint(2, 4), dtype="bf16",
                    layout=rng.choice(["tiled", "row_major"]), **rng.choice([WIDE, WIDE64]))
    if kind == "stats":
        return dict(kind="stats", T=_log_int(rng, 16, 16384), dtype="bf16", **rng.choice([WIDE, WIDE64, FEW]))
    shape = dict(rng.choice([WIDE, WIDE64, FEW]))
    recipe = rng.choice(["zero_bias", "zero_bias", "planted"])
    T = _log_int(rng, 1, 16384)
    if rng.random() < 0.2:  # the static layer, every slot on a normal expert
        shape["Z"], recipe, T = 0, "plain", min(T, 8192)
    return _layer(None, T, shape, layout=rng.choice(["tiled", "tiled", "row_major"]), gate=rng.choice(sorted(GATES)),
                  copy=rng.random() < 0.2, recipe=recipe)


# ---------------------------------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------------------------------
def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _planted(case, n, g, dev):
    """bool [n, N+Z], K entries per row: easy tokens (60 %) take 6-8 of 8 zero experts, hard ones 0-1 (in proportion for
    other K); normal experts are drawn without replacement by Zipf(1.1) popularity (exponential race)."""
    N, Z, K = case["N"], case["Z"], case["K"]
    easy = torch.rand(n, generator=g, device=dev) < 0.6
    u = torch.rand(n, generator=g, device=dev)
    zc = torch.where(easy, (0.75 * K + u * (0.25 * K + 1)).floor().clamp(max=K), (u * 2).floor()).long().clamp(max(0, K - N), min(K, Z))
    pop = torch.empty(N, device=dev)
    pop[torch.randperm(N, generator=g, device=dev)] = torch.arange(1, N + 1, device=dev, dtype=torch.float32) ** -1.1
    race = -torch.log(torch.rand(n, N, generator=g, device=dev).clamp_min(1e-30)) / pop
    plan = torch.zeros(n, N + Z, dtype=torch.bool, device=dev)
    plan[:, :N] = race.argsort(1).argsort(1) < (K - zc)[:, None]
    if Z:
        plan[:, N:] = torch.rand(n, Z, generator=g, device=dev).argsort(1).argsort(1) < zc[:, None]
    return plan


def _inputs(case, seed):
    dev, dt = torch.device("cuda"), _dtype(case)
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    T, H, I, N, Z, K = (case[k] for k in ("T", "H", "I", "N", "Z", "K"))
    recipe = case.get("recipe", "zero_bias")

    def normal(shape, std):
        return torch.randn(shape, generator=g, device=dev, dtype=torch.float32) * std

    wr = normal((N + Z, H), LOGIT_STD / math.sqrt(H))
    bias = None
    pool = T + T // 8 + 64
    x = normal((pool, H), 1.0)
    if recipe == "zero_bias":
        bias = torch.zeros(N + Z, device=dev)
        bias[N:] = ZERO_BIAS.get((N, Z, K), 0.5)
    elif recipe == "planted":
        # expert e owns one hidden coordinate: its router row is 3 there, a token of its plan carries 4, others 0
        coord = torch.randperm(H, generator=g, device=dev)[: N + Z]
        wr[torch.arange(N + Z, device=dev), coord] = 3.0
        x[:, coord] = torch.where(_planted(case, pool, g, dev), 4.0, 0.0)
    x, wr = x.to(dt), wr.to(dt)
    # Tokens whose selected set hangs on the last bits of a logit are left out, so that any two correct routers agree.
    top = torch.sort(_logits(x, wr, bias), dim=1, descending=True)
    ok = torch.ones(pool, dtype=torch.bool, device=dev)
    if K < N + Z:
        ok = top.values[:, K - 1] - top.values[:, K] > MIN_GAP
    if T == 1:
        ok &= (top.indices[:, :K] < N).any(1)  # a single token has work to do
    x = x[torch.nonzero(ok).view(-1)[:T]].contiguous()
    assert x.shape[0] == T
    out = {"x": x, "w_router": wr, "router_bias": bias}
    if case["kind"] == "layer":
        out["w_gate"] = normal((N, I, H), LOGIT_STD / math.sqrt(H)).to(dt)
        out["w_up"] = normal((N, I, H), LOGIT_STD / math.sqrt(H)).to(dt)
        out["w_down"] = normal((N, H, I), 0.55 / math.sqrt(I)).to(dt)
    return out


def _workload(case, seed):
    # (layer l of a stack draws from seed + l: seeds are spaced so that no two share a layer)
    return synth.Workload("stack", T=case["T"], H=case["H"], I=case["I"], N=case["N"], Z=case["Z"], K=case["K"], dtype=case["dtype"],
                          seed=64 * seed, recipe="zero_bias", zero_bias=ZERO_BIAS[(case["N"], case["Z"], case["K"])])


def _desc(case):
    layout = zeda.WEIGHTS_TILED if case.get("layout") == "tiled" else zeda.WEIGHTS_ROW_MAJOR
    return zeda.make_desc(case["T"], case["H"], case["I"], case["N"], case["Z"], case["K"], case["dtype"],
                          GATES[case.get("gate", "topk_norm")], layout, zeda.EXPERT_COPY if case.get("copy") else zeda.EXPERT_ZERO)


def prepare(case, seed):
    if case["kind"] == "stack":
        w = _workload(case, seed)
        x0 = synth.draw_tokens(w, "cuda")
        return {"kind": "stack", "stack": MoeStack(w, case["layers"], tiled=case["layout"] == "tiled"), "x0": x0, "x": x0.clone()}
    st = _inputs(case, seed)
    st["kind"], st["desc"] = case["kind"], _desc(case)
    if case["kind"] == "layer":
        if case["layout"] == "tiled":
            st["w_gate"], st["w_up"], st["w_down"] = zeda.zeda_pack_expert_weights(_desc(dict(case, layout="row_major")), st["w_gate"],
                                                                                    st["w_up"], st["w_down"])
        st["ws"] = torch.empty(zeda.workspace_bytes(st["desc"]), dtype=torch.uint8, device="cuda")
        st["out"] = torch.empty_like(st["x"])
        st["num_real"] = torch.zeros(1, dtype=torch.int32, device="cuda")
    return st


def run(st):
    if st["kind"] == "stack":
        return st["stack"].forward(st["x"].copy_(st["x0"]))  # the residual stream is updated in place
    if st["kind"] == "stats":
        return zeda.zeda_routing_stats(st["desc"], st["x"], st["w_router"], st["router_bias"], alpha=0.01, w=2.0)
    zeda.zeda_moe_forward(st["desc"], st["x"], st["w_router"], st["router_bias"], st["w_gate"], st["w_up"], st["w_down"], st["out"],
                          st["num_real"], st["ws"])
    return st["out"], st["num_real"]


def work(case):
    T, H, I, N, Z, K = (case[k] for k in ("T", "H", "I", "N", "Z", "K"))
    s = 2 if case["dtype"] == "bf16" else 4
    recipe = case.get("recipe", "zero_bias")
    zero = 0.0 if Z == 0 else Z / (N + Z) if recipe == "plain" else 0.55 if recipe == "planted" else 0.5
    R = T * K * (1.0 - zero)
    hit = N * (1.0 - (1.0 - 1.0 / N) ** R)  # experts with at least one row
    route_bytes, route_flops = (N + Z) * H * s + T * H * s, 2.0 * T * (N + Z) * H
    if case["kind"] == "stats":
        return {"bytes": route_bytes + 2.0 * (N + Z) * 4, "flops": route_flops}
    n = case.get("layers", 1)
    weights = n * (hit * 3 * H * I + (N + Z) * H) * s
    return {"bytes": weights + 2.0 * T * H * s, "flops": n * (route_flops + 6.0 * H * I * R)}


def tolerance(case):
    # about four times what the path shows against 64 bits: 3e-7 (statistics), 2e-7 (fp32 layer), 2.9e-3 (bf16 layer: the
    # roundings of the activations, of the expert outputs and of the result)
    if case["kind"] == "stats":
        return {"rel": 2e-6}
    if case["dtype"] == "f32":
        return {"rel": 1e-6}
    # (8e-3 for the residual stream after four layers, mostly the stream's own roundings, which two implementations share)
    return {"rel": 1.5e-2 if case["kind"] == "stack" else 1e-2}


# ---------------------------------------------------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------------------------------------------------
def _logits(x, wr, bias):
    lg = x.double() @ wr.double().t()
    return lg if bias is None else lg + bias.double()


def _top(logits, K):
    v, i = torch.sort(logits, dim=1, descending=True, stable=True)  # ties go to the lower index
    return v[:, :K], i[:, :K]


def _gates(logits, v, ids, N, gate):
    p = torch.softmax(logits, dim=1).gather(1, ids)
    if gate == "softmax":
        return p
    den = p.sum(1, keepdim=True) if gate == "topk_norm" else (p * (ids < N)).sum(1, keepdim=True)
    return torch.where(den > 0, p / den, torch.zeros_like(p))


def _moe(x, wr, bias, wg, wu, wd, N, K, gate, copy):
    logits = _logits(x, wr, bias)
    v, ids = _top(logits, K)
    gates = _gates(logits, v, ids, N, gate)
    x = x.double()
    out = torch.zeros_like(x)
    for e in range(N):
        tok, slot = torch.nonzero(ids == e, as_tuple=True)
        if tok.numel():
            h = x[tok]
            a = torch.nn.functional.silu(h @ wg[e].double().t()) * (h @ wu[e].double().t())
            out.index_add_(0, tok, (a @ wd[e].double().t()) * gates[tok, slot][:, None])
    if copy:
        out += (gates * (ids >= N)).sum(1, keepdim=True) * x
    return out, int((ids < N).sum())


def exact(case, seed):
    N, Z, K = case["N"], case["Z"], case["K"]
    if case["kind"] == "stack":
        w = _workload(case, seed)
        x = synth.draw_tokens(w, "cuda").double()
        for l in range(case["layers"]):
            wr, bias = synth.draw_router(w, "cuda", l)
            wg, wu, wd = synth.draw_experts(w, "cuda", l)
            xn = x / torch.sqrt((x * x).mean(1, keepdim=True) + EPS)
            x = x + _moe(xn, wr, bias, wg, wu, wd, N, K, "topk_norm", False)[0]
        return x
    L = _inputs(case, seed)
    if case["kind"] == "stats":
        logits = _logits(L["x"], L["w_router"], L["router_bias"])
        P = torch.softmax(logits, dim=1).mean(0)
        f = torch.zeros_like(logits).scatter_(1, _top(logits, K)[1], 1.0).mean(0)
        fE, PE, fZ, PZ = f[:N].sum(), P[:N].sum(), f[N:].sum(), P[N:].sum()
        la = 0.01 * (N + Z) / K * (f * P).sum()
        lga = 0.01 * (N + Z * 2.0) / K * (fE * PE / N + (fZ * PZ / (Z * 2.0) if Z else 0.0))
        return f, P, torch.stack([fE, PE, fZ, PZ, fZ / K, la, lga])
    out, real = _moe(L["x"], L["w_router"], L["router_bias"], L["w_gate"], L["w_up"], L["w_down"], N, K, case["gate"], case["copy"])
    return out, torch.tensor([real], dtype=torch.int64)
