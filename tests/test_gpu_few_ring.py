"""Row-major weights of few rows per expert go through LDS, tiled ones do not: the expert FFN gives the same bits for both, and the
right ones, where the reduction's chunks of 64 do not divide over the four waves, where a wave has one chunk, and for experts of
one to nine blocks of 16 rows, two or four of them a workgroup, with a dimension too short for it beside one that is not."""
import pytest

pytestmark = pytest.mark.gpu

from test_gpu_layout_bits import same_bits  # noqa: E402

# (T, K, Z, H, I, rows of every expert)
CASES = {
    "one_chunk_a_wave": (40, 1, 0, 256, 256, [1, 16, 17, 6]),
    "ragged_chunks": (60, 1, 2, 1152, 448, [1, 15, 16, 17, 2, 0, 9]),
    "deep": (20, 1, 0, 4096, 320, [3, 1, 0, 16]),
    "short_down": (64, 1, 0, 768, 128, [33, 31, 0]),
    "up_to_49_rows": (200, 1, 4, 1280, 704, [16, 33, 48, 49, 0, 1, 5, 40]),
    # (more slots per expert: four blocks of 16 rows a workgroup, of which one to four hold rows; two tiles for 65)
    "four_blocks": (320, 1, 0, 1280, 704, [33, 48, 49, 64, 65, 16, 1, 44]),
    "several_tiles": (400, 1, 0, 512, 256, [130, 33, 65, 64, 32, 76]),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_layouts_give_the_same_bits_for_few_rows(name):
    same_bits(*CASES[name])
