"""The statistics' final kernel has short loops for short calls and for rows of sums that are no whole 16-byte pieces, and wide ones from
7937 tokens on: the counts of both are those of the router's own ids, to the slot, and the probabilities' means those of 64 bits, on
both sides of that line and where the last block of 16 tokens, the last byte of a word of counts or the last word is the only one."""
import numpy as np
import pytest
import torch

from paper_2605_18643_amd import zeda

pytestmark = pytest.mark.gpu

POOLS = [(128, 32, 8), (20, 12, 4), (30, 7, 5), (200, 56, 16), (250, 3, 8)]


@pytest.mark.parametrize("pool", POOLS, ids=lambda p: "N%d_Z%d_K%d" % p)
@pytest.mark.parametrize("T", [1, 17, 256, 257, 4095, 7936, 7937, 8193])
def test_counts_and_means(T, pool):
    N, Z, K = pool
    H = 512
    print(T, pool, flush=True)
    g = torch.Generator(device="cuda").manual_seed(T + N)
    x = torch.randn(T, H, generator=g, device="cuda").bfloat16()
    wr = (torch.randn(N + Z, H, generator=g, device="cuda") * 0.9 / H ** 0.5).bfloat16()
    d = zeda.make_desc(T, H, 64, N, Z, K, "bf16")
    ids, gates = torch.empty(T, K, dtype=torch.int32, device="cuda"), torch.empty(T, K, device="cuda")
    ws = torch.empty(max(zeda.route_workspace_bytes(d), 16), dtype=torch.uint8, device="cuda")
    zeda.zeda_route(d, x, wr, None, ids, gates, ws=ws)
    f, P, summary = zeda.zeda_routing_stats(d, x, wr, None)
    torch.cuda.synchronize()
    counts = np.bincount(ids.cpu().numpy().ravel(), minlength=N + Z)
    assert (np.rint(f.cpu().numpy().astype(np.float64) * T) == counts).all()
    p = torch.softmax(x.double() @ wr.double().t(), 1).mean(0).cpu().numpy()
    # (logits of size up to five with sqrt(512) * 2^-24 of it as their error, 7e-6, in an exponent)
    np.testing.assert_allclose(P.cpu().numpy(), p, rtol=2e-5)
    np.testing.assert_allclose(summary.cpu().numpy()[[0, 2]], [counts[:N].sum() / T, counts[N:].sum() / T], rtol=1e-5, atol=1e-6)
