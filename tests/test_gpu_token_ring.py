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
