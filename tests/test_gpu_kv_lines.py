"""dK and dV on the lines between their kernels, against the oracle and against each other."""
import numpy as np
import pytest

from paper_2602_04789_amd import synth
from test_gpu_few_blocks import _check_head, _gradients, _lists
from test_gpu_parity import _dev, gpu  # noqa: F401

pytestmark = pytest.mark.gpu


# d = 64, past 256 KV blocks: lists of a few query blocks that are (nearly) all there are, and just not; d = 128, up to 128 KV blocks: mean lists
# of 48 and just below, of every query block; last blocks of 1, 31, 33 and 64 rows
@pytest.mark.parametrize("head_dim,heads,frame_len,per_chunk,frames,length", [
    (64, 111, 161, 1, 1, 3), (64, 53, 64, 3, 6, 3), (64, 44, 97, 2, 4, 4), (64, 32, 97, 5, 5, 4), (64, 44, 97, 2, 4, 3), (64, 39, 520, 1, 1, 7), (64, 32, 97, 5, 5, 7),
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



# 8 x 64 KV blocks with lists of 15 to 17 go to the general kernel, 9 x 64 to the one for long lists; the sums are in the same order.  Every KV
# block is kept by `kept` query blocks: odd and even numbers of half tiles.  (kept = 0) random lists, some ids out of range, two blocks that no
# list keeps, a query block without a valid id
@pytest.mark.parametrize("frame_len,kept", [(64, 15), (64, 16), (64, 17), (31, 15), (31, 16), (31, 17), (33, 16), (50, 17), (64, 0), (50, 0), (31, 0)])
def test_the_kernel_for_long_lists_has_the_bits_of_the_general_one(gpu, frame_len, kept):  # noqa: F811
    """Tensors carved out of larger ones; the first 8 heads the same bits in both calls and in repeated ones, heads against the oracle."""
    torch, lf = gpu
    heads, n_k, d = 9, 64, 128
    L = kept or 17
    assert 15 * n_k <= L * n_k < 18 * n_k and 512 < heads * n_k and (heads - 1) * n_k <= 512
    rng = np.random.default_rng(100 * frame_len + kept)
    x = {k: synth.f32_to_bf16_bits(rng.standard_normal((heads, n_k * frame_len, d), dtype=np.float32)) for k in ("Q", "K", "V", "dO")}
    if kept:
        lists = np.broadcast_to(np.sort((np.arange(n_k)[:, None] + np.arange(L)) % n_k, axis=1), (heads, n_k, L)).copy()
    else:
        ids = np.setdiff1d(np.arange(n_k), (5, n_k - 1))
        lists = np.stack([[np.sort(rng.choice(ids, L, replace=False)) for _ in range(n_k)] for _ in range(heads)])
        lists[:, ::3, 0], lists[:, ::2, -1] = -2, n_k + 3
        lists[1, 2] = n_k
    print(f"long lists and general kernel: frames of {frame_len}, {kept} query blocks a KV block", flush=True)

    def strided(bits, pad):
        view = torch.full((heads, bits.shape[1] + 3, d + pad), float("nan"), dtype=torch.bfloat16, device="cuda")[:, 1:-2, :d]
        view.copy_(_dev(torch, bits))
        return view
    Q, K, V, dO = (strided(x[k], p) for k, p in (("Q", 8), ("K", 16), ("V", 24), ("dO", 40)))
    idx = torch.from_numpy(lists.astype(np.int32)).cuda()
    out, lse2 = lf.lf_sparse_attn_fwd(Q, K, V, idx, frame_len, 64, O=torch.empty_strided(dO.shape, dO.stride(), dtype=dO.dtype, device="cuda"))

    def run(H):
        grads = tuple(torch.empty_strided(t[:H].shape, t.stride(), dtype=t.dtype, device="cuda").fill_(7.0) for t in (Q, K, V))
        lf.lf_sparse_attn_bwd(Q[:H], K[:H], V[:H], out[:H], dO[:H], lse2[:H], idx[:H], frame_len, 64, grads=grads)
        return grads
    long, general = run(heads), run(heads - 1)
    for name, a, b in zip(("dK", "dV"), long[1:], general[1:]):
        assert torch.equal(a[:-1].view(torch.int16), b.view(torch.int16)), name
    for _ in range(5):
        for a, b in zip(run(heads), long):
            assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    grads = [t.float().cpu().numpy().astype(np.float64) for t in long]
    if not kept:
        assert not grads[1][:, 5 * frame_len: 6 * frame_len].any() and not grads[2][:, -frame_len:].any()
    for h in (0, 1, heads - 1):
        _check_head(x, grads, lists, h, n_k, frame_len)
