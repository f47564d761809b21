"""dK and dV on the lines between their kernels, against the oracle."""
import numpy as np
import pytest

from test_gpu_few_blocks import _check_head, _gradients, _lists
from test_gpu_parity import gpu  # noqa: F401

pytestmark = pytest.mark.gpu


# d = 64, past 256 KV blocks: lists of a few query blocks that are (nearly) all there are, and just not; d = 128, up to 128 KV blocks: mean lists
# of 48 and just below, of every query block; last blocks of 1, 31, 33 and 64 rows
@pytest.mark.parametrize("head_dim,heads,frame_len,per_chunk,frames,length", [
    (64, 111, 161, 1, 1, 3), (64, 53, 64, 3, 6, 3), (64, 44, 97, 2, 4, 4), (64, 32, 97, 5, 5, 4), (64, 44, 97, 2, 4, 3),
    (128, 1, 64, 128, 128, 48), (128, 1, 64, 128, 128, 47), (128, 2, 33, 64, 64, 64), (128, 4, 31, 31, 32, 31), (128, 1, 65, 48, 64, 96)])
def test_gradients_on_the_lines_of_few_kv_blocks(gpu, head_dim, heads, frame_len, per_chunk, frames, length):  # noqa: F811
    torch, lf = gpu
    nb = -(-frame_len // 64)
    rng = np.random.default_rng(heads + length)
    lists = _lists(rng, heads, per_chunk * nb, frames * nb, length)
    print(f"lines of few KV blocks: {heads * frames * nb} d={head_dim} n={frame_len} list length {length}", flush=True)
    x, grads = _gradients(torch, lf, rng, heads, frame_len, per_chunk, frames, head_dim, lists)
    for h in {0, heads - 1}:
        _check_head(x, grads, lists, h, frames * nb, frame_len)
