"""fp32 kernels at the sizes where a tile, a k step or a block of experts ends: whole-layer parity with the oracle."""
import numpy as np
import pytest
import torch

from oracle import harness
from paper_2605_18643_amd import synth, zeda

pytestmark = pytest.mark.gpu

from gpu_util import forward, full_parity  # noqa: E402

CASES = [
    # k tails of 4 and 28 past whole 32-wide chunks, feature tails of 4 and 12, more k slices than chunks
    dict(T=33, H=132, I=20, N=3, Z=2, K=2),
    dict(T=70, H=60, I=44, N=4, Z=0, K=1),
    dict(T=1, H=4, I=4, N=2, Z=1, K=2),
    # experts with about 16 / 32 / 33 / 64 rows (token blocks of 16, tiles of 32)
    dict(T=64, H=96, I=64, N=4, Z=0, K=1),
    dict(T=130, H=256, I=128, N=4, Z=0, K=1),
    dict(T=300, H=64, I=36, N=9, Z=3, K=3),
    # expert counts on both sides of 16, 32, 64 and 128 (router blocks), and the wide feature tile (N * 2I, N * H >= 16384)
    dict(T=40, H=100, I=16, N=17, Z=0, K=4),
    dict(T=20, H=72, I=16, N=40, Z=25, K=5),
    dict(T=50, H=1028, I=524, N=33, Z=7, K=6),
    dict(T=37, H=68, I=8, N=120, Z=9, K=16),
    dict(T=17, H=128, I=8, N=160, Z=96, K=8),
]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: "_".join(f"{k}{v}" for k, v in c.items()))
def test_f32_layer_at_tile_edges(cfg):
    w = synth.Workload("f32_tiles", dtype="f32", seed=301, recipe="plain", x_std=1.0, w_std=0.05, wr_std=0.05, **cfg)
    print(w, flush=True)
    full_parity(w, harness.gapped_layer(w, "cuda"))


def test_f32_infinities_stay_infinite():
    """One infinite hidden value: every product with it is an infinity, and so are the sums it enters (no NaN from the
    sum's own bookkeeping); tokens without it are untouched."""
    w = synth.Workload("f32_inf", T=40, H=256, I=64, N=4, Z=0, K=1, dtype="f32", seed=302, recipe="plain", x_std=1.0, w_std=0.05, wr_std=0.05)
    L = harness.gapped_layer(w, "cuda")
    d = zeda.make_desc(w.T, w.H, w.I, w.N, w.Z, w.K, "f32")
    base = forward(w, L)
    off, ss = base["expert_offsets"].cuda(), base["sorted_slot"].cuda()
    x = L["x"].clone()
    x[7, 5] = float("inf")
    y = torch.empty((w.T * w.K, w.H), device="cuda")
    ws = torch.empty(zeda.expert_ffn_workspace_bytes(d), dtype=torch.uint8, device="cuda")
    zeda.zeda_expert_ffn(d, x, L["w_gate"], L["w_up"], L["w_down"], off, ss, base["num_real"].cuda(), y, ws)
    torch.cuda.synchronize()
    act = ws[: w.T * w.I * 4].view(torch.float32).view(w.T, w.I).cpu()
    row = int(base["slot_to_row"][7])
    e = int(base["topk_ids"][7, 0])
    g, u = L["w_gate"][e, :, 5].cpu(), L["w_up"][e, :, 5].cpu()
    # silu(+inf) * (+-inf) = +-inf; silu(-inf) = -inf / inf = NaN, as plain fp32 arithmetic has it
    want_inf = (g > 0) & (u != 0)
    assert torch.equal(act[row][want_inf], torch.where(u > 0, np.inf, -np.inf).to(torch.float32)[want_inf])
    others = torch.ones(w.T, dtype=torch.bool)
    others[row] = False
    assert torch.equal(y.cpu()[others], base["y_slot"][others])


def test_f32_more_token_tiles_than_one_grid_row():
    """More than 16384 tiles of 32 rows: the launch continues along the grid's second dimension.  Expert FFN alone, every
    row against float64."""
    N, H, I, T = 2, 4, 4, 540000
    g = torch.Generator().manual_seed(11)
    x = torch.randn(T, H, generator=g)
    wg, wu = torch.randn(N, I, H, generator=g), torch.randn(N, I, H, generator=g)
    wd = torch.randn(N, H, I, generator=g)
    n0 = 270001
    off = torch.tensor([0, n0, T], dtype=torch.int32)
    slots = torch.arange(T, dtype=torch.int32)
    d = zeda.make_desc(T, H, I, N, 0, 1, "f32")
    y = torch.full((T, H), float("nan"), device="cuda")
    ws = torch.empty(zeda.expert_ffn_workspace_bytes(d), dtype=torch.uint8, device="cuda")
    zeda.zeda_expert_ffn(d, x.cuda(), wg.cuda(), wu.cuda(), wd.cuda(), off.cuda(), slots.cuda(), off[2:].cuda(), y, ws)
    torch.cuda.synchronize()
    for e, (a, b) in enumerate([(0, n0), (n0, T)]):
        h = x[a:b].double()
        ref = (torch.nn.functional.silu(h @ wg[e].double().t()) * (h @ wu[e].double().t())) @ wd[e].double().t()
        got = y[a:b].cpu().double()
        assert (got - ref).norm() <= 1e-5 * ref.norm() and (got - ref).abs().max() <= 1e-5 * ref.abs().max()


def test_chunk_sums_that_cancel():
    """The running sums keep what an addition rounds off, also where the summand is the larger one: 2^28 comes and goes
    between summands below one, which survive to fp32 accuracy.  (One product per 32-wide chunk, so that the sums within a
    chunk are exact; whatever chunk a slice of 16 starts with, a small sum meets 2^28 in it.)"""
    H, slices, per = 4096, 16, 8
    g = torch.Generator().manual_seed(9)
    big = 2.0 ** 28
    pattern = torch.tensor([0.0, big, -big, 0.0, big, -big, 0.0, 0.0])
    small = torch.rand(per, slices, generator=g) * (pattern == 0)[:, None] / slices
    wr = torch.zeros(2, H)
    wr[0, ::32] = (pattern[:, None] + small).flatten()  # chunk i * slices + s is the i-th of slice s
    x = torch.ones(3, H)
    d = zeda.make_desc(3, H, 64, 2, 0, 2, "f32")
    ids = torch.full((3, 2), -1, dtype=torch.int32, device="cuda")
    gates = torch.empty((3, 2), device="cuda")
    zeda.zeda_route(d, x.cuda(), wr.cuda(), None, ids, gates)
    torch.cuda.synchronize()
    logit = small.double().sum()
    assert logit > 1 and (ids.cpu() == torch.tensor([0, 1], dtype=torch.int32)).all()
    # (16 slices of four errors, added in fp32: within 1e-6)
    np.testing.assert_allclose(gates.cpu().double().numpy()[:, 0], float(1 / (1 + torch.exp(-logit))), rtol=2e-6)
