"""Expert GEMM tiles with the 64-wide token ring: shortest reductions (fewer pairs of chunks than the ring holds), ragged
tiles, both sides of the rule that chooses it; parity with the oracle, and the bits of the row-major path."""
import numpy as np
import pytest
import torch

from oracle import harness
from paper_2605_18643_amd import synth

pytestmark = pytest.mark.gpu

from gpu_util import full_parity  # noqa: E402

CASES = [
    dict(T=700, H=256, I=128, N=8, Z=0, K=2),     # down: two pairs of chunks, nothing but the tail part; 175 rows
    dict(T=1209, H=512, I=128, N=44, Z=0, K=4),   # one slot short of 110 per expert ...
    dict(T=1210, H=512, I=128, N=44, Z=0, K=4),   # ... and exactly there
    dict(T=1300, H=768, I=384, N=24, Z=4, K=3),   # odd numbers of pairs; several items per workgroup
    dict(T=3000, H=256, I=256, N=30, Z=10, K=2),
    dict(T=5000, H=256, I=384, N=16, Z=0, K=2),   # 625 rows: several token tiles per expert
]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: "_".join(f"{k}{v}" for k, v in c.items()))
def test_token_ring_matches_the_oracle_and_the_row_major_path(cfg):
    w = synth.Workload("ring", dtype="bf16", seed=501, recipe="plain", x_std=1.0, w_std=min(0.05, 0.9 * cfg["H"] ** -0.5), wr_std=0.05, **cfg)
    print(w, flush=True)
    L = harness.gapped_layer(w, "cuda")
    tokens = np.arange(0, w.T, 9)
    plain, _ = full_parity(w, L, tokens=tokens)
    tiled, _ = full_parity(w, L, tokens=tokens, tiled=True)
    assert torch.equal(plain["out"].view(torch.int16), tiled["out"].view(torch.int16))


@pytest.mark.parametrize("Z", [0, 10], ids=["wide_ring", "narrow_ring"])
@pytest.mark.parametrize("tiled", [False, True], ids=["row_major", "tiled"])
def test_expert_loads_around_32_row_blocks(Z, tiled):
    """Experts with 1, 31, 32, 33, ... rows: the second wave row leaves out a last block that holds no rows.  Expert FFN
    alone against float64 (bf16 rounding of the activations and of the result: 2^-9 each, relative)."""
    from paper_2605_18643_amd import zeda

    loads = [1, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 160, 161, 192, 193, 224, 225, 256, 257]
    N, H, I = len(loads), 256, 384
    T = sum(loads)
    g = torch.Generator().manual_seed(7)
    x = torch.randn(T, H, generator=g).bfloat16()
    wg, wu = ((torch.randn(N, I, H, generator=g) * H ** -0.5).bfloat16() for _ in range(2))
    wd = (torch.randn(N, H, I, generator=g) * I ** -0.5).bfloat16()
    off = torch.tensor(np.concatenate([[0], np.cumsum(loads)]), dtype=torch.int32)
    slots = torch.randperm(T, generator=g).to(torch.int32)
    d = zeda.make_desc(T, H, I, N, Z, 1, "bf16", weight_layout=zeda.WEIGHTS_TILED if tiled else zeda.WEIGHTS_ROW_MAJOR)
    W = [t.cuda() for t in (wg, wu, wd)]
    if tiled:
        W = zeda.zeda_pack_expert_weights(zeda.make_desc(T, H, I, N, Z, 1, "bf16"), *W)
    y = torch.full((T, H), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(zeda.expert_ffn_workspace_bytes(d), dtype=torch.uint8, device="cuda")
    zeda.zeda_expert_ffn(d, x.cuda(), *W, off.cuda(), slots.cuda(), off[N:].cuda(), y, ws)
    torch.cuda.synchronize()
    for e in range(N):
        r0, r1 = int(off[e]), int(off[e + 1])
        h = x[slots[r0:r1].long()].double()
        a = torch.nn.functional.silu(h @ wg[e].double().t()) * (h @ wu[e].double().t())
        ref = a @ wd[e].double().t()
        rel = (y[r0:r1].cpu().double() - ref).norm(dim=1) / ref.norm(dim=1)
        assert rel.max() < 1e-2, (e, loads[e], float(rel.max()))
