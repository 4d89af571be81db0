"""Short slot lists, which the gate/up kernels place themselves (and for which, up to four tokens, they select too): the tables that a
whole-layer call leaves against zeda_dispatch on its ids, bit for bit, at both ends of what they take, and the layer against the oracle."""
import numpy as np
import pytest
import torch

from oracle import harness
from paper_2605_18643_amd import synth, zeda

pytestmark = pytest.mark.gpu

from gpu_util import forward, full_parity  # noqa: E402


def _layer(dtype, T, N, Z, K, **kw):
    # sizes of the few-row kernel for any load (few weight tiles), and of the fp32 kernels.  Weights of 0.02 at H = 2048: the absolute
    # tolerance of bf16 layers (2e-2) is for outputs below two, which half a last place of bf16 (2^-9) leaves a factor of five
    base = dict(H=2048, I=128) if dtype == "bf16" else dict(H=100, I=36)
    return synth.Workload("tile_place", T=T, N=N, Z=Z, K=K, dtype=dtype, seed=701, recipe="zero_bias", x_std=1.0, w_std=0.02, wr_std=0.02 if dtype == "bf16" else 0.05,
                          zero_bias=kw.pop("zero_bias", 0.3), **base)


def _check_tables(w, L):
    """Everything that later kernels read, as zeda_dispatch has it for the same ids."""
    res = forward(w, L)
    d = zeda.make_desc(w.T, w.H, w.I, w.N, w.Z, w.K, w.dtype)
    ids = res["topk_ids"].cuda()
    S = w.T * w.K
    off, ss, s2r, nr = (torch.full((n,), -9, dtype=torch.int32, device="cuda") for n in (w.N + 1, S, S, 1))
    ws = torch.empty(zeda.dispatch_workspace_bytes(d), dtype=torch.uint8, device="cuda")
    zeda.zeda_dispatch(d, ids, off, ss, s2r, nr, ws)
    torch.cuda.synchronize()
    R = int(nr)
    assert int(res["num_real"]) == R == res["num_real_out"]
    assert torch.equal(res["expert_offsets"], off.cpu()) and torch.equal(res["slot_to_row"], s2r.cpu())
    assert torch.equal(res["sorted_slot"][:R], ss.cpu()[:R])
    return res


# one slot; on both sides of four tokens; whole and ragged groups of 64 slots; 1024 slots and one token more
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("shape", [(1, 3, 2, 1), (1, 20, 12, 16), (2, 30, 9, 8), (4, 33, 7, 5), (4, 40, 0, 16), (5, 33, 7, 5), (16, 20, 12, 4),
                                   (65, 7, 3, 1), (146, 24, 8, 7), (128, 40, 4, 8), (129, 40, 4, 8), (1024, 12, 5, 1), (1025, 12, 5, 1)],
                         ids=lambda s: "T%d_N%d_Z%d_K%d" % s)
def test_tables_of_short_lists(dtype, shape):
    w = _layer(dtype, *shape)
    print(w, flush=True)
    full_parity(w, harness.gapped_layer(w, "cuda"))
    _check_tables(w, harness.gapped_layer(w, "cuda"))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T", [3, 200])
def test_one_hot_expert_and_no_real_slot(dtype, T):
    """All slots on one expert, several token tiles; none on any, so that no tile exists."""
    for bias_at, real in ((5, True), (9, False)):
        w = _layer(dtype, T, 8, 4, 1)
        L = harness.gapped_layer(w, "cuda")
        L["router_bias"] = torch.zeros(12, device="cuda")
        L["router_bias"][bias_at] = 100.0
        res = _check_tables(w, L)
        assert res["num_real_out"] == (T if real else 0)
        if not real:
            assert not res["out"].float().any()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T", [4, 40])
def test_tokens_without_an_expert(dtype, T):
    """A token of no-numbers gets no expert: its slots are placed nowhere, the others are as without it."""
    w = _layer(dtype, T, 24, 8, 4)
    L = harness.gapped_layer(w, "cuda")
    x = L["x"].clone()
    x[1] = float("nan")
    res = _check_tables(w, dict(L, x=x))
    base = forward(w, L)
    assert (res["topk_ids"][1] == np.iinfo(np.int32).max).all()
    keep = torch.arange(T) != 1
    assert torch.equal(res["topk_ids"][keep], base["topk_ids"][keep]) and torch.equal(res["topk_gates"][keep], base["topk_gates"][keep])
    assert not res["out"][1].float().any()


# the number of workgroups from which on the slots get a launch of their own: 6960 and 7424 (bound 7168), 3456 and 3600 (bound 3500)
BOUND_CASES = [("bf16", 256, 960, 100), ("bf16", 256, 1024, 100), ("f32", 64, 768, 128), ("f32", 64, 800, 128)]


@pytest.mark.parametrize("dtype,H,I,N", BOUND_CASES)
def test_tables_on_both_sides_of_the_workgroup_bound(dtype, H, I, N):
    w = synth.Workload("tile_place", T=64, H=H, I=I, N=N, Z=30, K=8, dtype=dtype, seed=702, recipe="zero_bias", x_std=1.0, w_std=0.02, wr_std=0.05,
                       zero_bias=0.1)
    print(w, flush=True)
    full_parity(w, harness.gapped_layer(w, "cuda"))
    _check_tables(w, harness.gapped_layer(w, "cuda"))
