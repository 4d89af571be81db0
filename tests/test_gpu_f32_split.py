"""fp32 expert FFN of many rows per expert (numbers as sums of three bf16 parts): whole-layer parity with the oracle where a tile, a
k chunk or a slice of the waves ends, and rows with elements that have no such sum."""
import numpy as np
import pytest
import torch

from oracle import harness
from paper_2605_18643_amd import synth, zeda

pytestmark = pytest.mark.gpu

from gpu_util import full_parity  # noqa: E402

# all wide (N * 2I and N * H at least 16384) with eight slots per expert or more
CASES = [
    # experts with about 16, 32, 33 and 90 rows; chunks that the slices of the four waves do not divide; fewer chunks than slices
    dict(T=128, H=1024, I=512, N=16, Z=0, K=2),
    dict(T=130, H=2048, I=1024, N=8, Z=2, K=2),
    dict(T=264, H=1024, I=512, N=16, Z=0, K=2),
    dict(T=360, H=2052, I=1028, N=8, Z=0, K=2),
    # k tails of 4 and 28, feature tails of 4 and 12
    dict(T=70, H=1060, I=516, N=32, Z=3, K=5),
    dict(T=64, H=156, I=92, N=110, Z=0, K=14),
]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: "_".join(f"{k}{v}" for k, v in c.items()))
def test_f32_split_layer_at_tile_edges(cfg):
    w = synth.Workload("f32_split", dtype="f32", seed=311, recipe="plain", x_std=1.0, w_std=0.05, wr_std=0.05, **cfg)
    print(w, flush=True)
    full_parity(w, harness.gapped_layer(w, "cuda"))


def _ffn(d, x, wg, wu, wd, off, slots):
    y = torch.full((d.T * d.K, d.H), float("nan"), device="cuda")
    ws = torch.empty(zeda.expert_ffn_workspace_bytes(d), dtype=torch.uint8, device="cuda")
    zeda.zeda_expert_ffn(d, x, wg, wu, wd, off, slots, off[-1:], y, ws)
    torch.cuda.synchronize()
    return ws[: d.T * d.I * 4].view(torch.float32).view(d.T, d.I).cpu(), y.cpu()


def test_f32_split_huge_elements():
    """Elements that a bf16 rounds to infinity, in a token and in a weight row: what depends on them is what 64-bit sums give,
    everything else keeps its bits."""
    T, H, I, N = 160, 2048, 1024, 8
    g = torch.Generator().manual_seed(12)
    x = torch.randn(T, H, generator=g)
    wg, wu = 0.05 * torch.randn(N, I, H, generator=g), 0.05 * torch.randn(N, I, H, generator=g)
    wd = 0.05 * torch.randn(N, H, I, generator=g)
    off = (torch.arange(N + 1) * (T // N)).to(torch.int32).cuda()
    slots = torch.arange(T, dtype=torch.int32, device="cuda")
    d = zeda.make_desc(T, H, I, N, 0, 1, "f32")
    act0, y0 = _ffn(d, x.cuda(), wg.cuda(), wu.cuda(), wd.cuda(), off, slots)
    # token 7 (expert 0, second block of 16 from row 16 on: token 17 too), a gate row of expert 3 and a down row of expert 5
    x[7, 5], x[17, 2040], wg[3, 100, 9], wd[5, 77, 1000] = float("inf"), 3.39e38, float("-inf"), 3.3999e38
    act, y = _ffn(d, x.cuda(), wg.cuda(), wu.cuda(), wd.cuda(), off, slots)
    e = torch.arange(T) // (T // N)
    want = act0.clone()
    for t in (7, 17):
        gg, uu = ((x[t].double() @ m[e[t]].double().t()).float() for m in (wg, wu))
        want[t] = gg / (1 + torch.exp(-gg)) * uu
    rows = e == 3
    gg, uu = (x[rows].double() @ wg[3, 100].double()).float(), (x[rows].double() @ wu[3, 100].double()).float()
    want[rows, 100] = gg / (1 + torch.exp(-gg)) * uu
    changed = torch.zeros_like(act, dtype=torch.bool)
    changed[[7, 17]] = True
    changed[rows, 100] = True
    assert torch.equal(act[~changed], act0[~changed])
    # (sums of 2048 products in another order of the 64-bit additions, then expf and a division: a few last places)
    np.testing.assert_allclose(act[changed].numpy(), want[changed].numpy(), rtol=2e-6)
    assert torch.isinf(act[7]).any() and not torch.isnan(act[17]).any()
    # the down projection: row 77 of expert 5's weights, and the tokens whose activations changed
    same = torch.ones_like(y, dtype=torch.bool)
    same[[7, 17]] = False
    same[rows] = False
    same[e == 5, 77] = False
    assert torch.equal(y[same], y0[same])
    ref = (act[e == 5].double() @ wd[5, 77].double()).float()
    np.testing.assert_allclose(y[e == 5, 77].numpy(), ref.numpy(), rtol=2e-6)
