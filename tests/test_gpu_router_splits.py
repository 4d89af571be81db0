"""The bf16 router where the hidden dimension is split over workgroups and a second kernel selects, and where it is not, for both
workgroup sizes: ids, gates, placement and statistics against the oracle.  How many slices ran is read off the scratch, so
that a case cannot stop reaching the kernels it is here for.  (zeda_route and the statistics run the second kernel; whole-layer
calls of few slots place, and up to four tokens select, in the gate/up kernel.  Its own placement: test_gpu_place_list.)"""
import ctypes

import numpy as np
import pytest
import torch

from oracle import harness, zeda_oracle as orc
from paper_2605_18643_amd import synth, zeda

pytestmark = pytest.mark.gpu

from gpu_util import check_dispatch, check_routing, desc_of, forward  # noqa: E402

GATES = [zeda.GATE_SOFTMAX, zeda.GATE_TOPK_NORM, zeda.GATE_REAL_RENORM]
FILL, GUARD = 0xA5, 4096


def _scratch(nbytes):
    return torch.full((nbytes + GUARD,), FILL, dtype=torch.uint8, device="cuda")


def _slices(d, ws, nbytes):
    """Slices whose logits are in the scratch: [slice][tokens, whole blocks of 16][experts, whole blocks of 32] from its
    start; nothing else is written (the bytes that stay as they were are those of a fresh buffer)."""
    b = ws.cpu().numpy()
    table = -(-d.T // 16) * 16 * (-(-(d.N + d.Z) // 32) * 32) * 4
    written = np.flatnonzero(b != FILL)
    n = 0 if written.size == 0 else -(-(int(written[-1]) + 1) // table)
    assert n * table <= nbytes and (b[n * table:] == FILL).all()
    return n


# (T, H, N, Z, K, slices)
CASES = [
    # 16 waves: eight slices; both sides of the 16 tokens of a selecting workgroup; sixteen slices
    (1, 2048, 128, 32, 8, 8),
    (9, 2048, 128, 32, 8, 8),
    (16, 2048, 128, 32, 16, 8),
    (17, 2048, 128, 32, 8, 8),
    (100, 2048, 70, 27, 6, 8),
    (3, 4096, 100, 28, 4, 16),
    (40, 4096, 200, 56, 8, 8),
    # four and two slices, ragged last blocks; two slices of 32-token blocks
    (513, 2048, 128, 32, 8, 4),
    (1030, 2048, 128, 64, 8, 2),
    (2041, 2048, 128, 32, 8, 2),
    (2500, 4096, 200, 56, 4, 2),
    # one kernel, with 16, 32 and 64 tokens a workgroup
    (203, 1024, 70, 27, 6, 0),
    (2500, 512, 128, 32, 8, 0),
    (5000, 256, 128, 32, 8, 0),
    (16500, 128, 70, 26, 3, 0),
    # four waves: splits, a full and a ragged selecting workgroup, one kernel with 16, 32 and 64 tokens a workgroup
    (1, 2048, 24, 8, 2, 8),
    (16, 2048, 20, 12, 16, 8),
    (17, 2048, 40, 24, 4, 8),
    (5, 4096, 10, 3, 3, 16),
    (700, 4096, 24, 8, 4, 8),
    (1501, 7168, 33, 20, 4, 4),
    (3001, 4096, 40, 20, 4, 2),
    (300, 512, 24, 8, 4, 0),
    (6001, 512, 24, 8, 4, 0),
    (16400, 128, 20, 6, 2, 0),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "T%d_H%d_N%d_Z%d_K%d_s%d" % c)
def test_router_splits_match_the_oracle(case):
    T, H, N, Z, K, slices = case
    gate = GATES[(T + N) % 3]
    w = synth.Workload("splits", T=T, H=H, I=64, N=N, Z=Z, K=K, dtype="bf16", seed=601, recipe="zero_bias", x_std=1.0, w_std=0.02,
                       wr_std=2.0 * H ** -0.5, zero_bias=0.3)
    print(w, gate, flush=True)
    L = harness.gapped_layer(w, "cuda", gate_norm=gate)
    a = harness.to_arrays(L)
    rid, rg, logits = orc.route(a["x"], a["w_router"], a["router_bias"], N, Z, K, gate, want_logits=True)
    d, top = desc_of(w, gate), float(np.max(np.abs(logits)))

    nbytes = zeda.route_workspace_bytes(d)
    ws = _scratch(nbytes)
    ids = torch.full((T, K), -1, dtype=torch.int32, device="cuda")
    gates = torch.full((T, K), float("nan"), device="cuda")
    zeda.zeda_route(d, L["x"], L["w_router"], L["router_bias"], ids, gates, ws=ws[:max(nbytes, 16)])
    torch.cuda.synchronize()
    check_routing(w, {"topk_ids": ids.cpu(), "topk_gates": gates.cpu()}, rid, rg, top)
    assert _slices(d, ws, nbytes) == slices

    # the whole layer: the same ids and gates, and the placement that starts from them
    res = forward(w, L, gate)
    check_routing(w, res, rid, rg, top)
    check_dispatch(w, res, rid)

    # the statistics: the same kernels, with the routing probabilities of every block
    f, P, _ = zeda.zeda_routing_stats(d, L["x"], L["w_router"], L["router_bias"], alpha=0.01, w=2.0)
    torch.cuda.synchronize()
    ref = orc.routing_stats(a["x"], a["w_router"], a["router_bias"], N, Z, K, alpha=0.01, w=2.0)
    np.testing.assert_allclose(f.cpu().numpy().astype(np.float64), ref["f"], rtol=1e-6, atol=1e-7)
    # (a probability's relative error is the error of a difference of two logits, as a gate's is)
    np.testing.assert_allclose(P.cpu().numpy().astype(np.float64), ref["P"], rtol=2e-5 + 2.0 * np.sqrt(H) * 2.0 ** -24 * top, atol=1e-7)


def test_statistics_scratch_is_not_overrun():
    """Expert counts that are no multiple of four and ragged token blocks, with exactly the bytes that the query returns."""
    for dtype, H in (("bf16", 2048), ("f32", 68)):
        for T, N, Z in ((33, 29, 4), (70, 128, 31), (300, 5, 2)):
            g = torch.Generator().manual_seed(T)
            tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
            x, wr = torch.randn(T, H, generator=g).to(tdt).cuda(), (0.05 * torch.randn(N + Z, H, generator=g)).to(tdt).cuda()
            d = zeda.make_desc(T, H, 64, N, Z, 3, dtype)
            nbytes = int(zeda.lib().zeda_routing_stats_workspace_bytes(ctypes.byref(d)))
            ws = _scratch(nbytes)
            f, P, s = (torch.full((n,), float("nan"), device="cuda") for n in (N + Z, N + Z, 7))
            rc = zeda.lib().zeda_routing_stats(ctypes.byref(d), x.data_ptr(), wr.data_ptr(), None, 0.01, 2.0, f.data_ptr(), P.data_ptr(),
                                               s.data_ptr(), ws.data_ptr(), nbytes, None)
            torch.cuda.synchronize()
            assert rc == zeda.ZEDA_OK and (ws[nbytes:].cpu() == FILL).all()
            p = torch.softmax(x.double() @ wr.double().t(), dim=1)
            np.testing.assert_allclose(P.cpu().double().numpy(), p.mean(0).cpu().numpy(), rtol=2e-4)
            assert abs(float(f.sum()) - 3.0) < 1e-5
