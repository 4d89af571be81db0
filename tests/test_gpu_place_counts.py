"""The placement that starts from the router's per-block counts, and the statistics' sums, at the token counts where the way of
reading the counts changes (12 words of 16 blocks, 16, 32, 64 lanes to an expert's words): tables against zeda_dispatch on the
same ids, bit for bit, and statistics against 64 bits."""
import numpy as np
import pytest
import torch

from paper_2605_18643_amd import zeda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,Z", [(1, 2), (40, 9), (128, 32), (250, 6)])
@pytest.mark.parametrize("T", [2900, 3072, 3073, 4096, 4097, 8192, 8200, 16384])
def test_tables_and_statistics(T, N, Z):
    K, H, I = 2, 128, 64
    g = torch.Generator(device="cuda").manual_seed(T + N)
    x = torch.randn(T, H, generator=g, device="cuda").bfloat16()
    wr = (torch.randn(N + Z, H, generator=g, device="cuda") * 2 / H ** 0.5).bfloat16()
    w = [torch.zeros(s, dtype=torch.bfloat16, device="cuda") for s in ((N, I, H), (N, I, H), (N, H, I))]
    d = zeda.make_desc(T, H, I, N, Z, K, "bf16")
    ws = torch.full((zeda.workspace_bytes(d),), 0xA5, dtype=torch.uint8, device="cuda")
    out, nr = torch.empty_like(x), torch.zeros(1, dtype=torch.int32, device="cuda")
    zeda.zeda_moe_forward(d, x, wr, None, *w, out, nr, ws)
    v = zeda.ws_views(d, ws)
    off, ss, s2r, r = (torch.full((n,), -9, dtype=torch.int32, device="cuda") for n in (N + 1, T * K, T * K, 1))
    dws = torch.empty(zeda.dispatch_workspace_bytes(d), dtype=torch.uint8, device="cuda")
    zeda.zeda_dispatch(d, v["topk_ids"].contiguous(), off, ss, s2r, r, dws)
    torch.cuda.synchronize()
    R = int(r)
    assert int(nr) == R == int(v["num_real"]) and torch.equal(v["expert_offsets"], off) and torch.equal(v["slot_to_row"], s2r)
    assert torch.equal(v["sorted_slot"][:R], ss[:R])
    f, P, _ = zeda.zeda_routing_stats(d, x, wr, None)
    torch.cuda.synchronize()
    assert torch.equal(torch.round(f.double() * T).long(), torch.bincount(v["topk_ids"].flatten().long(), minlength=N + Z))
    p = torch.softmax(x.double() @ wr.double().t(), dim=1).mean(0)
    # (each probability to a few last places of fp32 and of its logits' 2^-24 sqrt(H) |logit|; errors of the mean are smaller)
    np.testing.assert_allclose(P.double().cpu().numpy(), p.cpu().numpy(), rtol=2e-5)
