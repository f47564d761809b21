"""lf_sparse_attn_split on both sides of the line between one pass and a dense phase over a long current chunk."""
import numpy as np
import pytest

from oracle import hsa_oracle as O
from paper_2602_04789_amd import synth
from test_gpu_parity import MAX_ABS, MEAN_ABS, _dev, _host_f32, gpu  # noqa: F401

pytestmark = pytest.mark.gpu


# A chunk of 199 and 200 blocks; 768 and 769 or more query blocks at d = 64, 1 024 and more at d = 128; at d = 128 a last round of
# 699 blocks (dense phase) and of 700 (one pass); frames with a last block of 1, 33 and 64 rows; lists without a retrieved block
@pytest.mark.parametrize("head_dim,heads,frame_len,per_chunk,keep", [
    (64, 4, 64, 199, 5), (64, 4, 64, 200, 5), (64, 4, 97, 100, 0), (64, 3, 64, 256, 9), (64, 5, 65, 101, 70), (128, 5, 64, 200, 3),
    (128, 6, 64, 200, 5), (128, 6, 97, 100, 31), (128, 4, 65, 128, 4), (128, 5, 65, 103, 0), (128, 8, 64, 215, 6), (128, 8, 64, 216, 33)])
def test_the_split_call_on_long_chunks(gpu, head_dim, heads, frame_len, per_chunk, keep):  # noqa: F811
    torch, lf = gpu
    nb, hist = -(-frame_len // 64), 75
    frames, n_q, n_k = hist + per_chunk, per_chunk * nb, (hist + per_chunk) * nb
    rng = np.random.default_rng(heads * per_chunk + keep)
    mk = lambda t: synth.f32_to_bf16_bits(rng.standard_normal((heads, t * frame_len, head_dim), dtype=np.float32))
    x = {"Q": mk(per_chunk), "K": mk(frames), "V": mk(frames)}
    lists = np.empty((heads, n_q, keep + n_q), dtype=np.int32)
    for h in range(heads):
        for r in range(n_q):
            lists[h, r, :keep] = np.sort(rng.permutation(hist * nb)[:keep])
    lists[:, :, keep:] = np.arange(hist * nb, n_k)
    b = lf.lf_budget()
    b.n_hist_frames, b.frames_per_chunk, b.k_frames, b.k_blocks = hist, per_chunk, hist, keep
    b.current_mandatory, b.list_len, b.keep_ratio = 1, keep + n_q, 0.5
    print(f"split call: d={head_dim} {heads * n_q} query blocks, {n_q} current blocks, {keep} retrieved", flush=True)
    Q, K, V = (_dev(torch, x[k]) for k in "QKV")
    idx = torch.from_numpy(lists).cuda()
    one = lf.lf_sparse_attn(Q, K, V, idx, frame_len, 64)
    idx[:, :, keep:] = -3                      # not read
    runs = [lf.lf_sparse_attn_split(Q, K, V, idx, frame_len, 64, b) for _ in range(2)]
    torch.cuda.synchronize()
    assert torch.equal(runs[0].view(torch.int16), runs[1].view(torch.int16))
    diff = (one.float() - runs[0].float()).abs()
    assert float(diff.max()) <= 2 * MAX_ABS and float(diff.mean()) <= 2 * MEAN_ABS
    got = runs[0].float().cpu().numpy().astype(np.float64)
    for h, r in ((0, 0), (heads - 1, n_q - 1), (heads // 2, nb - 1), (1, n_q // 2)):
        lo, hi = O.block_token_range(r, frame_len, 64)
        ref = O.sparse_attention_block(*(_host_f32(x[k][h]) for k in "QKV"), r, [int(c) for c in lists[h, r]], frame_len, 64)
        err = np.abs(got[h, lo:hi] - ref)
        assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS, (h, r, err.max(), err.mean())
