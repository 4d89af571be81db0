"""A whole-layer call of a handful of tokens selects in the gate/up kernel, zeda_route in the router's second kernel (of four waves up to
64 experts, of sixteen beyond): ids and gates have the same bits, on both sides of the four tokens, of the 64 experts and of the 1024
workgroups from which on the gate/up kernel leaves the selection to the router."""
import pytest
import torch

from oracle import harness
from paper_2605_18643_amd import synth, zeda

pytestmark = pytest.mark.gpu

from gpu_util import desc_of, forward  # noqa: E402

GATES = [zeda.GATE_SOFTMAX, zeda.GATE_TOPK_NORM, zeda.GATE_REAL_RENORM]


# H: such that the router is split over the hidden dimension (eight or sixteen slices).  I = 2688: 1008 workgroups, 2752: 1032
SHAPES = [(1, 24, 8, 2, 2048, 64), (2, 5, 2, 3, 4096, 64), (4, 40, 24, 6, 2048, 64), (3, 33, 20, 4, 4096, 64), (4, 20, 12, 16, 2048, 64),
          (5, 40, 24, 6, 2048, 64), (1, 60, 5, 4, 2048, 64), (4, 128, 32, 8, 2048, 64), (3, 200, 56, 8, 4096, 64), (1, 40, 24, 6, 2048, 2688),
          (1, 40, 24, 6, 2048, 2752), (1, 128, 32, 6, 2048, 2752)]


@pytest.mark.parametrize("gate", GATES)
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "T%d_N%d_Z%d_K%d_H%d_I%d" % s)
def test_layer_and_router_select_alike(shape, gate):
    T, N, Z, K, H, I = shape
    w = synth.Workload("select_bits", T=T, H=H, I=I, N=N, Z=Z, K=K, dtype="bf16", seed=811, recipe="zero_bias", x_std=1.0, w_std=0.02,
                       wr_std=2.0 * H ** -0.5, zero_bias=0.3)
    print(w, gate, flush=True)
    L = harness.gapped_layer(w, "cuda", gate_norm=gate)
    d = desc_of(w, gate)
    ids, gates = torch.full((T, K), -1, dtype=torch.int32, device="cuda"), torch.full((T, K), float("nan"), device="cuda")
    ws = torch.empty(max(zeda.route_workspace_bytes(d), 16), dtype=torch.uint8, device="cuda")
    zeda.zeda_route(d, L["x"], L["w_router"], L["router_bias"], ids, gates, ws=ws)
    torch.cuda.synchronize()
    res = forward(w, L, gate)
    assert torch.equal(res["topk_ids"], ids.cpu())
    assert torch.equal(res["topk_gates"].view(torch.int32), gates.cpu().view(torch.int32))
