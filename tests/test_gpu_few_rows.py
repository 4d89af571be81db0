"""The expert FFN of small batches and small models, and the router's splits, at the sizes where a tile, a slice or a rule
ends: whole-layer parity with the oracle in both weight layouts, whose results are the same bits."""
import numpy as np
import pytest
import torch

from oracle import harness
from paper_2605_18643_amd import synth

pytestmark = pytest.mark.gpu

from gpu_util import full_parity  # noqa: E402

CASES = [
    # one token; a reduction dimension with fewer 64-wide chunks than waves; one expert
    dict(T=1, H=128, I=64, N=3, Z=1, K=2),
    dict(T=1, H=2048, I=768, N=128, Z=32, K=8),
    dict(T=7, H=256, I=192, N=1, Z=0, K=1),
    # about 16, 17, 32 and 33 rows per expert (token blocks of 16, tiles of 32), several tiles per expert
    dict(T=64, H=384, I=64, N=4, Z=0, K=1),
    dict(T=130, H=1152, I=448, N=4, Z=0, K=1),
    dict(T=200, H=640, I=320, N=8, Z=2, K=2),
    # both sides of the rules, in slots per expert of the pool: 170 (next to no weight tiles), 40 and 30 (four token blocks a
    # workgroup, few weight tiles), 25 to 26 (two blocks to four), 13 (one full round of the chip), 5 (more than that)
    dict(T=2720, H=128, I=64, N=14, Z=2, K=1),
    dict(T=2721, H=128, I=64, N=14, Z=2, K=1),
    dict(T=320, H=1280, I=704, N=12, Z=4, K=2),
    dict(T=321, H=1280, I=704, N=12, Z=4, K=2),
    dict(T=341, H=1152, I=448, N=24, Z=8, K=3),
    dict(T=342, H=1152, I=448, N=24, Z=8, K=3),
    dict(T=200, H=1152, I=448, N=24, Z=0, K=3),
    dict(T=201, H=1152, I=448, N=24, Z=0, K=3),
    dict(T=208, H=768, I=512, N=60, Z=4, K=4),
    dict(T=209, H=768, I=512, N=60, Z=4, K=4),
    dict(T=100, H=768, I=1024, N=100, Z=60, K=8),
    dict(T=101, H=768, I=1024, N=100, Z=60, K=8),
    dict(T=80, H=768, I=1088, N=64, Z=0, K=4),
    dict(T=81, H=768, I=1088, N=64, Z=0, K=4),
    # both sides of 8 slots per expert (weights of experts with several token tiles kept in the caches or not)
    dict(T=128, H=768, I=512, N=30, Z=2, K=2),
    dict(T=129, H=768, I=512, N=30, Z=2, K=2),
    # decode batches: three and four live token blocks; both sides of the rule beyond which the 64-row tile takes over; a
    # reduction too short for the waves
    dict(T=50, H=1024, I=1024, N=8, Z=0, K=6),
    dict(T=64, H=512, I=512, N=16, Z=0, K=16),
    dict(T=50, H=768, I=1024, N=50, Z=0, K=8),
    dict(T=51, H=768, I=1024, N=50, Z=0, K=8),
    dict(T=64, H=512, I=256, N=200, Z=20, K=8),
    # both sides of the 16 tokens of the router's selecting workgroups, widest pool, slots on every expert
    dict(T=16, H=2048, I=64, N=60, Z=30, K=16),
    dict(T=17, H=2048, I=64, N=60, Z=30, K=16),
    dict(T=33, H=1024, I=64, N=200, Z=56, K=4),
    dict(T=1, H=1024, I=64, N=5, Z=251, K=16),
]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: "_".join(f"{k}{v}" for k, v in c.items()))
def test_small_batches_match_the_oracle_in_both_layouts(cfg):
    # (weights scaled with the widths so that outputs keep the magnitude the absolute bound is meant for: 0.02 at H = 2048)
    w = synth.Workload("few", dtype="bf16", seed=401, recipe="plain", x_std=1.0, w_std=min(0.05, 0.9 * cfg["H"] ** -0.5), wr_std=0.05, **cfg)
    print(w, flush=True)
    L = harness.gapped_layer(w, "cuda")
    tokens = None if w.T <= 400 else np.arange(0, w.T, 5)
    plain, _ = full_parity(w, L, tokens=tokens)
    tiled, _ = full_parity(w, L, tokens=tokens, tiled=True)
    assert torch.equal(plain["out"].view(torch.int16), tiled["out"].view(torch.int16))


@pytest.mark.parametrize("T", [4096, 4097, 8192, 8193, 8250, 16390])
def test_router_splits_of_long_batches(T):
    """One workgroup per 16, 32 and 64 tokens, the last one partly filled, through the per-block counts that the placement
    starts from: ids, gates, placement and output of sampled tokens.  160 experts: 16 waves; 64: four."""
    for N, Z in ((128, 32), (40, 24)):
        w = synth.Workload("route_long", T=T, H=256, I=64, N=N, Z=Z, K=5, dtype="bf16", seed=402, recipe="zero_bias", x_std=1.0,
                           w_std=0.05, wr_std=0.08, zero_bias=0.3)
        print(w, flush=True)
        full_parity(w, harness.gapped_layer(w, "cuda"), tokens=np.arange(0, T, 37))


def test_masked_experts_are_not_selected_twice():
    """Experts masked with a bias of -inf: the others come first, then masked ones, each once, with weight zero."""
    from paper_2605_18643_amd import zeda

    for T in (5, 300, 5000):
        for dtype, H in (("bf16", 256), ("f32", 64)):
            g = torch.Generator().manual_seed(T)
            tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
            N, Z, K = 20, 4, 6
            x, wr = torch.randn(T, H, generator=g).to(tdt).cuda(), (0.1 * torch.randn(N + Z, H, generator=g)).to(tdt).cuda()
            bias = torch.full((N + Z,), float("-inf"))
            keep = [3, 8, 17, 22]
            bias[keep] = 0.0
            ids = torch.full((T, K), -1, dtype=torch.int32, device="cuda")
            gates = torch.full((T, K), float("nan"), device="cuda")
            d = zeda.make_desc(T, H, 64, N, Z, K, dtype)
            ws = torch.empty(max(16, zeda.route_workspace_bytes(d)), dtype=torch.uint8, device="cuda")
            zeda.zeda_route(d, x, wr, bias.cuda(), ids, gates, ws=ws)
            torch.cuda.synchronize()
            i, gt = ids.cpu().numpy(), gates.cpu().numpy()
            assert (np.sort(i[:, :4], axis=1) == keep).all() and (i[:, 4:] == [0, 1]).all()
            assert (gt[:, 4:] == 0).all() and np.allclose(gt.sum(1), 1.0, atol=1e-5)


@pytest.mark.parametrize("dtype,H", [("bf16", 256), ("bf16", 1024), ("f32", 64)])
@pytest.mark.parametrize("N,Z", [(20, 4), (70, 27)])
def test_statistics_count_masked_experts_once(dtype, H, N, Z):
    """f_i (Eq. 4) of experts masked with a bias of -inf: the selected slots of the router itself."""
    from paper_2605_18643_amd import zeda

    for T in (5, 300):
        g = torch.Generator().manual_seed(T)
        tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
        K, NE = 6, N + Z
        x, wr = torch.randn(T, H, generator=g).to(tdt).cuda(), (0.1 * torch.randn(NE, H, generator=g)).to(tdt).cuda()
        bias = torch.full((NE,), float("-inf"))
        bias[[3, 8, 17, 22]] = 0.0
        d = zeda.make_desc(T, H, 64, N, Z, K, dtype)
        f, P, _ = zeda.zeda_routing_stats(d, x, wr, bias.cuda())
        ids = torch.full((T, K), -1, dtype=torch.int32, device="cuda")
        zeda.zeda_route(d, x, wr, bias.cuda(), ids, torch.empty((T, K), device="cuda"))
        torch.cuda.synchronize()
        counts = np.bincount(ids.cpu().numpy().ravel(), minlength=NE)
        assert np.array_equal(f.cpu().numpy(), (counts / T).astype(np.float32))
        assert f.max() <= 1 and np.allclose(f.cpu().numpy()[[0, 1]], 1.0)
        np.testing.assert_allclose(P.cpu().numpy().sum(), 1.0, rtol=1e-5)


@pytest.mark.parametrize("dtype,H,N", [("bf16", 2048, 90), ("bf16", 256, 90), ("bf16", 256, 20), ("f32", 64, 20)])
def test_experts_without_a_logit_leave_the_other_gates_alone(dtype, H, N):
    """Fewer than K experts have a logit that is a number: those come first, with the gates that they have among
    themselves, and the remaining slots weigh nothing."""
    from paper_2605_18643_amd import zeda

    for T in (5, 300):
        g = torch.Generator().manual_seed(T)
        tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
        K, Z = 6, 4
        x, wr = torch.randn(T, H, generator=g).to(tdt).cuda(), (0.02 * torch.randn(N + Z, H, generator=g)).to(tdt).cuda()
        bias = torch.full((N + Z,), float("nan"))
        keep = [3, 8, 17, N + 2]
        bias[keep] = 0.0
        for norm in (zeda.GATE_TOPK_NORM, zeda.GATE_REAL_RENORM):
            d = zeda.make_desc(T, H, 64, N, Z, K, dtype, gate_norm=norm)
            ids = torch.full((T, K), -1, dtype=torch.int32, device="cuda")
            gates = torch.full((T, K), float("nan"), device="cuda")
            ws = torch.empty(max(16, zeda.route_workspace_bytes(d)), dtype=torch.uint8, device="cuda")
            zeda.zeda_route(d, x, wr, bias.cuda(), ids, gates, ws=ws)
            torch.cuda.synchronize()
            i, gt = ids.cpu().numpy(), gates.cpu().numpy()
            assert (np.sort(i[:, :4], axis=1) == keep).all() and (gt[:, 4:] == 0).all()
            logit = np.take_along_axis((x.double() @ wr.double().T).cpu().numpy(), i[:, :4], 1)
            ex = np.exp(logit - logit.max(1, keepdims=True))
            real = np.ones_like(ex) if norm == zeda.GATE_TOPK_NORM else i[:, :4] < N
            # (fp32 logits of up to H = 2048 products of |x w| of about 0.016: within 1e-4)
            np.testing.assert_allclose(gt[:, :4], ex / (ex * real).sum(1, keepdims=True), rtol=5e-4)
