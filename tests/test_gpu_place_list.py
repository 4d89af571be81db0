"""Calls of up to 16 tokens whose experts the few-row kernel does not take: the router's second kernel selects and places, with four
waves (up to 64 experts) and with sixteen, for whole and ragged groups of 64 slots.  (test_dispatch_rules holds the cases to that.)"""
import numpy as np
import pytest
import torch

from oracle import harness
from paper_2605_18643_amd import synth, zeda

pytestmark = pytest.mark.gpu

from gpu_util import full_parity  # noqa: E402

# (T, H, I, N, Z, K)
CASES = [
    (16, 2048, 256, 40, 8, 8),
    (13, 2048, 256, 40, 8, 7),
    (5, 2048, 256, 40, 8, 16),
    (16, 2048, 256, 40, 24, 16),
    (7, 4096, 256, 44, 4, 11),
    (16, 2048, 64, 128, 32, 16),
    (11, 2048, 256, 128, 32, 13),
    (9, 2048, 256, 100, 30, 15),
    (16, 4096, 256, 200, 56, 16),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "T%d_H%d_I%d_N%d_Z%d_K%d" % c)
def test_router_places(case):
    T, H, I, N, Z, K = case
    w = synth.Workload("place_list", T=T, H=H, I=I, N=N, Z=Z, K=K, dtype="bf16", seed=821, recipe="zero_bias", x_std=1.0, w_std=0.9 * H ** -0.5,
                       wr_std=2.0 * H ** -0.5, zero_bias=0.3)
    print(w, flush=True)
    for gate in (zeda.GATE_SOFTMAX, zeda.GATE_TOPK_NORM):
        full_parity(w, harness.gapped_layer(w, "cuda", gate_norm=gate), gate)


@pytest.mark.parametrize("case", [CASES[0], CASES[5]], ids=lambda c: "T%d_H%d_I%d_N%d_Z%d_K%d" % c)
def test_router_places_no_real_slot_and_tokens_without_an_expert(case):
    T, H, I, N, Z, K = case
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn(T, H, generator=g, device="cuda").bfloat16()
    wr = (torch.randn(N + Z, H, generator=g, device="cuda") * 2 / H ** 0.5).bfloat16()
    w = [torch.zeros(s, dtype=torch.bfloat16, device="cuda") for s in ((N, I, H), (N, I, H), (N, H, I))]
    bias = torch.zeros(N + Z, device="cuda")
    bias[N:] = 1000.0  # (K <= Z: every slot on a zero expert)
    x[1] = float("nan")
    for b in ((bias, None) if K <= Z else (None,)):
        d = zeda.make_desc(T, H, I, N, Z, K, "bf16")
        ws = torch.full((zeda.workspace_bytes(d),), 0xA5, dtype=torch.uint8, device="cuda")
        out, nr = torch.full_like(x, 7.0), torch.full((1,), -1, dtype=torch.int32, device="cuda")
        zeda.zeda_moe_forward(d, x, wr, b, *w, out, nr, ws)
        v = zeda.ws_views(d, ws)
        off, ss, s2r, r = (torch.full((n,), -9, dtype=torch.int32, device="cuda") for n in (N + 1, T * K, T * K, 1))
        dws = torch.empty(zeda.dispatch_workspace_bytes(d), dtype=torch.uint8, device="cuda")
        zeda.zeda_dispatch(d, v["topk_ids"].contiguous(), off, ss, s2r, r, dws)
        torch.cuda.synchronize()
        R = int(r)
        assert (R == 0) == (b is not None) and int(nr) == R == int(v["num_real"])
        assert torch.equal(v["expert_offsets"], off) and torch.equal(v["slot_to_row"], s2r) and torch.equal(v["sorted_slot"][:R], ss[:R])
        assert (v["topk_ids"][1] == np.iinfo(np.int32).max).all() and not out.float().any()
