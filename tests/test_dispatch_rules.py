"""Which kernels a whole-layer call takes, by the library's rules on the host: both sides of the bounds on placing and selecting in the
gate/up kernel, and the paths that the GPU tests' cases are there for."""
import importlib

import pytest

from paper_2605_18643_amd import zeda

import dispatch_rules as rules


def _desc(T, H, I, N, Z, K, dtype="bf16"):
    return zeda.make_desc(T, H, I, N, Z, K, dtype)


def _workgroups(T, I, N, K, rows, cols):
    S = T * K
    return (min(S, N) + S // rows) * -(-I // cols)


@pytest.mark.parametrize("H,bound", [(256, 7168), (1024, 7168), (2048, 14336), (4096, 28672)])
def test_placing_is_bounded_by_workgroups(H, bound):
    seen = set()
    for T, K in ((1, 16), (5, 8), (32, 4), (64, 8), (64, 16), (65, 8), (128, 8), (129, 8)):
        for N in (16, 64, 128, 240):
            for I in (64, 512, 768, 1024, 1536, 2048, 4096):
                d = _desc(T, H, I, N, 8, K)
                nb = rules.few_blocks(d)
                want = nb > 0 and T * K <= 1024 and _workgroups(T, I, N, K, 16 * nb, 16) <= bound
                assert rules.gateup_places(d) == want, (T, H, I, N, K)
                seen.add((nb > 0, want))
    assert {(True, True), (True, False)} <= seen


@pytest.mark.parametrize("H,bound", [(256, 3500), (1024, 3500), (2044, 3500), (2048, 9216), (4096, 18432)])
def test_placing_of_fp32_layers_is_bounded_by_workgroups(H, bound):
    for T, K in ((1, 16), (64, 8), (64, 16), (129, 8)):
        for N in (4, 64, 128, 240):
            for I in (36, 512, 1024, 4096):
                wide = N * 2 * I >= 16384
                want = T * K <= 1024 and _workgroups(T, I, N, K, 32, 32 if wide else 16) <= bound
                assert rules.gateup_places(_desc(T, H, I, N, 8, K, "f32")) == want, (T, H, I, N, K)


def test_selecting_is_bounded_by_tokens_and_workgroups():
    for T in (1, 2, 4, 5):
        for K in (2, 8, 16):
            for I in (64, 768, 1536, 2688, 2752, 4096):
                d = _desc(T, 2048, I, 128, 32, K)
                want = T <= 4 and rules.few_blocks(d) == 2 and _workgroups(T, I, 128, K, 32, 16) <= 1024
                assert rules.gateup_selects(d) == want, (T, K, I)
    # the cases of the benchmark: one token selects there, 32 and 64 place there
    assert rules.gateup_selects(_desc(1, 2048, 768, 128, 32, 8))
    assert all(rules.gateup_places(_desc(T, 2048, 768, 128, Z, 8)) and not rules.gateup_selects(_desc(T, 2048, 768, 128, Z, 8)) for T, Z in ((32, 64), (64, 32)))


def test_gpu_cases_take_the_paths_they_are_there_for():
    place = importlib.import_module("test_gpu_place_list")
    for T, H, I, N, Z, K in place.CASES:
        d = _desc(T, H, I, N, Z, K)
        assert rules.whole_layer_places(d) == "router" and rules.few_blocks(d) == 0
    ring = importlib.import_module("test_gpu_few_ring")
    blocks = {n: rules.few_blocks(_desc(c[0], c[3], c[4], len(c[5]), c[2], c[1])) for n, c in ring.CASES.items()}
    assert blocks["four_blocks"] == 4 and set(blocks.values()) == {2, 4}
    tables = importlib.import_module("test_gpu_tile_place")
    sides = [rules.gateup_places(_desc(64, H, I, N, 30, 8, t)) for t, H, I, N in tables.BOUND_CASES]
    assert sides == [True, False, True, False]
    select = importlib.import_module("test_gpu_select_bits")
    selects = [rules.gateup_selects(_desc(T, H, I, N, Z, K)) for T, N, Z, K, H, I in select.SHAPES]
    assert all(rules.route_splits(_desc(T, H, I, N, Z, K)) for T, N, Z, K, H, I in select.SHAPES)
    assert {(s, N + Z > 64) for s, (T, N, Z, K, H, I) in zip(selects, select.SHAPES)} == {(True, False), (True, True), (False, False), (False, True)}
