"""lf_sparse_attn_split on both sides of its line: a dense phase over the current chunk whose state the list-driven kernel goes on
from, or one pass.  Which one ran shows in the workspace, which only the dense phase writes."""
import numpy as np
import pytest

from oracle import hsa_oracle as O
from paper_2602_04789_amd import synth
from test_gpu_parity import MAX_ABS, MEAN_ABS, _dev, _host_f32, gpu  # noqa: F401

pytestmark = pytest.mark.gpu


# In two phases: frames with last blocks of 1, 8, 33 and 36 rows, both head dimensions, lists without and with many retrieved blocks.  In one
# pass: 256 query blocks and fewer, whole frames, a chunk that saves less than the state costs.  (kind) plain: unit normal inputs;
# retrieved, current: those blocks' scores far above the others, in both orders of the carried state and what follows it
@pytest.mark.parametrize("head_dim,heads,frame_len,per_chunk,keep,two,kind,scale", [
    (64, 27, 97, 15, 7, True, "plain", 0.0), (64, 27, 97, 15, 7, True, "retrieved", 1.0), (64, 27, 97, 15, 7, True, "current", 4.0),
    (64, 17, 65, 24, 0, True, "plain", 0.0), (64, 11, 200, 20, 60, True, "retrieved", 4.0), (64, 20, 33, 40, 33, True, "plain", 0.25),
    (128, 22, 97, 30, 20, True, "plain", 0.0), (128, 22, 97, 30, 20, True, "retrieved", 1.0), (128, 22, 97, 30, 20, True, "current", 1.0),
    (128, 11, 65, 30, 5, True, "retrieved", 4.0), (128, 17, 200, 20, 0, True, "plain", 0.0), (128, 14, 100, 20, 3, True, "retrieved", 0.25),
    (64, 8, 97, 16, 7, False, "retrieved", 1.0), (64, 13, 64, 60, 7, False, "plain", 0.0), (128, 5, 64, 225, 31, False, "current", 1.0),
    (128, 24, 200, 6, 40, False, "retrieved", 1.0)])
def test_the_split_call_on_both_sides_of_its_line(gpu, head_dim, heads, frame_len, per_chunk, keep, two, kind, scale):  # noqa: F811
    """Tensors carved out of larger ones, entries of the current chunk unread, the same bits in a second call, sampled blocks against
    the oracle."""
    torch, lf = gpu
    nb, hist = -(-frame_len // 64), 40
    frames, n_q, n_k = hist + per_chunk, per_chunk * nb, (hist + per_chunk) * nb
    rng = np.random.default_rng(heads * per_chunk + keep)

    def strided(tokens, pad_tok, pad_ch, factor=None):
        x = rng.standard_normal((heads, tokens, head_dim), dtype=np.float32)
        if factor is not None:
            x *= factor[None, :, None]
        bits = synth.f32_to_bf16_bits(x)
        buf = torch.full((heads, tokens + pad_tok, head_dim + pad_ch), float("nan"), dtype=torch.bfloat16, device="cuda")
        view = buf[:, 1:1 + tokens, :head_dim]
        view.copy_(_dev(torch, bits))
        return buf, view, _host_f32(bits)
    hist_tok = hist * frame_len
    low, high = {"plain": (1.0, 1.0), "retrieved": (3.0, 0.05), "current": (0.05, 3.0)}[kind]
    factor = np.where(np.arange(frames * frame_len) < hist_tok, np.float32(low), np.float32(high)).astype(np.float32)
    (_, Q, Qf), (_, K, Kf), (_, V, Vf) = strided(per_chunk * frame_len, 3, 8), strided(frames * frame_len, 2, 24, factor), strided(frames * frame_len, 4, 16)
    Obuf, Oview, _ = strided(per_chunk * frame_len, 5, 40)
    Obuf.fill_(float("nan"))
    lists = np.empty((heads, n_q, keep + n_q), dtype=np.int32)
    for h in range(heads):
        for r in range(n_q):
            lists[h, r, :keep] = np.sort(rng.permutation(hist * nb)[:keep])
    lists[:, :, keep:] = np.arange(hist * nb, n_k)
    unread = lists.copy()
    unread[:, :, keep:] = -3
    b = lf.lf_budget()
    b.n_hist_frames, b.frames_per_chunk, b.k_frames, b.k_blocks = hist, per_chunk, hist, keep
    b.current_mandatory, b.list_len, b.keep_ratio = 1, keep + n_q, 0.5
    print(f"split call: d={head_dim} n={frame_len} {heads * n_q} query blocks, {n_q} current and {keep} retrieved, {kind}", flush=True)
    idx = torch.from_numpy(unread).cuda()
    ws = torch.full((lf.lf_attn_workspace_bytes(lf.make_shape(Q, K, V, Oview, frame_len, 64)),), 0xA5, dtype=torch.uint8, device="cuda")
    out = lf.lf_sparse_attn_split(Q, K, V, idx, frame_len, 64, b, softmax_scale=scale, O=Oview, workspace=ws)
    assert bool((ws != 0xA5).any()) == two
    again = lf.lf_sparse_attn_split(Q, K, V, idx, frame_len, 64, b, softmax_scale=scale)
    assert torch.equal(out.contiguous().view(torch.int16), again.view(torch.int16))
    got = out.float().cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all()
    for h, r in ((0, 0), (heads - 1, n_q - 1), (heads // 2, nb - 1), (1, n_q // 2), (heads - 2, 1)):
        lo, hi = O.block_token_range(r, frame_len, 64)
        ref = O.sparse_attention_block(Qf[h], Kf[h], Vf[h], r, [int(c) for c in lists[h, r]], frame_len, 64, scale=scale or None)
        err = np.abs(got[h, lo:hi] - ref)
        assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS, (h, r, err.max(), err.mean())
    tokens = per_chunk * frame_len
    assert torch.isnan(Obuf[:, :1].float()).all() and torch.isnan(Obuf[:, 1 + tokens:].float()).all()
    assert torch.isnan(Obuf[:, :, head_dim:].float()).all()
