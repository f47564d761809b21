"""The attention kernel with two wavefronts per query block and undivided lists at d = 128, which takes calls of 449 to 512 query blocks past a full
round of 1 024, and calls of more than 512 with lists of fewer than 16 (V asked for early in whole frames up to 1 024)."""
import pytest

import test_gpu_parity as parity
from test_gpu_parity import gpu  # noqa: F401

pytestmark = pytest.mark.gpu


# 1 536 query blocks (whole and short frames, lists of 32) and, lists of 12: 528 of whole frames, 528 of short ones
@pytest.mark.parametrize("scale", [0.25, 1.0, 4.0])
@pytest.mark.parametrize("frame_len,heads,chunk", [(200, 192, 4), (256, 192, 4), (192, 88, 2), (161, 88, 2)])
def test_the_reference_moves_inside_undivided_lists(gpu, frame_len, heads, chunk, scale):  # noqa: F811
    parity.test_extreme_logits_with_many_query_blocks(gpu, frame_len, 128, heads, chunk, scale)


def test_undivided_lists_around_the_decode_passes(gpu):  # noqa: F811
    """1 536 query blocks with lists around one and two passes of 256 entries."""
    parity.test_list_lengths_around_the_decode_passes(gpu, 384, (255, 256, 257, 513), 128)
