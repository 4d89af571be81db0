"""Both weight layouts add in the same order: the expert FFN gives the same bits for row-major and for tiled weights under
loads that make the kernels choose differently - one tile per expert (items start at k chunks of their own), several tiles
with a low mean, loads where the 320-row geometry (tiled only) saves passes over the weights."""
import numpy as np
import pytest
import torch

from paper_2605_18643_amd import zeda

pytestmark = pytest.mark.gpu

# (T, K, Z, H, I, rows of every expert)
# (wide enough for the tile kernels: more than 40 tiles of 128 columns of I over all experts)
CASES = {
    # 300 rows take one 320-row tile and two 256-row ones: the tiled path takes the wider geometry, at a mean of 144 / 120 rows
    "wide_tile_low_mean": (2304, 1, 8, 512, 768, [300, 300, 300, 50, 50, 50, 50, 50]),
    "wide_tile_few_hot": (2304, 1, 8, 768, 896, [300, 300, 60, 60, 60, 60, 60, 60]),
    "wide_tile_all": (2304, 1, 0, 512, 768, [288] * 8),
    # one tile per expert, both ends of the region with start chunks of their own; several tiles inside it
    "even_63": (700, 1, 3, 2048, 768, [63] * 6 + [0, 0]),
    "even_64": (700, 1, 3, 2048, 768, [64] * 6 + [0, 0]),
    "even_191": (1530, 1, 0, 1024, 768, [191] * 8),
    "even_192": (1536, 1, 0, 1024, 768, [192] * 8),
    "hot_in_region": (2400, 1, 4, 1024, 768, [700, 70, 80, 90, 60, 100, 50, 64]),
    # widths that only the narrow tile divides; many rows
    "narrow": (1600, 1, 2, 1152, 832, [150, 120, 90, 200, 256, 64, 100, 140]),
    "many_rows": (9000, 1, 0, 512, 768, [1100, 1200, 900, 1000, 1300, 800, 1400, 1300]),
}
# token rows of more than 4 GiB, of the activations and of x, read by 32-bit offsets no more: tiles of 256 rows, of 320 rows,
# and loads at which there is no choice between them
BIG_CASES = {
    "act_256": (131088, 1, 0, 256, 16384, [512] * 256),
    "act_320": (131088, 1, 0, 256, 16384, [560] * 234 + [2] * 22),
    "act_many_rows": (131088, 1, 0, 256, 16384, [2048] * 63 + [2064]),
    "x_256": (131088, 1, 0, 16384, 128, [512] * 256),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_layouts_give_the_same_bits(name):
    same_bits(*CASES[name])


@pytest.mark.parametrize("name", sorted(BIG_CASES))
def test_layouts_give_the_same_bits_above_4_gib_of_token_rows(name):
    T, K, Z, H, I, loads = BIG_CASES[name]
    assert T * K * max(I, H) * 2 > 2 ** 32
    same_bits(*BIG_CASES[name], stride=61)


def draw(shape, scale, g):
    t = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    for part in t.split(max(1, (1 << 27) // (t[0].numel()))):
        part.copy_(torch.randn(part.shape, generator=g, device="cuda") * scale)
    return t


def same_bits(T, K, Z, H, I, loads, stride=1):
    """stride: of the experts whose rows are also compared with float64 (the last one always is)"""
    N, R = len(loads), sum(loads)
    print(T, H, I, loads, flush=True)
    g = torch.Generator("cuda").manual_seed(T + H)
    x = draw((T, H), 1.0, g)
    wg, wu = (draw((N, I, H), H ** -0.5, g) for _ in range(2))
    wd = draw((N, H, I), I ** -0.5, g)
    off = torch.tensor(np.concatenate([[0], np.cumsum(loads)]), dtype=torch.int32).cuda()
    slots = torch.randperm(T * K, generator=g, device="cuda")[:R].to(torch.int32)
    out = []
    for layout in (zeda.WEIGHTS_ROW_MAJOR, zeda.WEIGHTS_TILED):
        d = zeda.make_desc(T, H, I, N, Z, K, "bf16", weight_layout=layout)
        W = (wg, wu, wd) if layout == zeda.WEIGHTS_ROW_MAJOR else zeda.zeda_pack_expert_weights(zeda.make_desc(T, H, I, N, Z, K, "bf16"), wg, wu, wd)
        y = torch.full((T * K, H), float("nan"), dtype=torch.bfloat16, device="cuda")
        ws = torch.empty(zeda.expert_ffn_workspace_bytes(d), dtype=torch.uint8, device="cuda")
        zeda.zeda_expert_ffn(d, x, *W, off, slots, off[N:], y, ws)
        torch.cuda.synchronize()
        out.append(y[:R].cpu())
        del y, ws, W
    assert torch.equal(out[0].view(torch.int16), out[1].view(torch.int16))
    # and they are the right ones: float64 on a few rows of every expert (bf16 rounding of activations and result)
    for e, (a, m) in enumerate(zip(np.cumsum([0] + loads[:-1]), loads)):
        if e % stride and e != N - 1:
            continue
        r = torch.arange(a, a + m, max(1, m // 7))
        h = x[(slots[r] // K).long()].cpu().double()
        act = torch.nn.functional.silu(h @ wg[e].cpu().double().t()) * (h @ wu[e].cpu().double().t())
        ref = act @ wd[e].cpu().double().t()
        assert m == 0 or ((out[0][r].double() - ref).norm(dim=1) / ref.norm(dim=1)).max() < 1e-2, e
