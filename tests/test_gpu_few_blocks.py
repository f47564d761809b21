"""Calls with few query or KV blocks, whose row halves get workgroups of their own, against the oracle."""
import numpy as np
import pytest

from oracle import hsa_oracle as O
from paper_2602_04789_amd import synth
from test_gpu_attn_bwd import _close
from test_gpu_parity import MAX_ABS, MEAN_ABS, _dev, _host_f32, gpu  # noqa: F401

pytestmark = pytest.mark.gpu


def _lists(rng, heads, n_q, n_k, length):
    """Ascending lists with ids out of range at both ends, some with few valid ids or none."""
    lists = np.full((heads, n_q, length), n_k + 1, dtype=np.int64)
    for h in range(heads):
        for r in range(n_q):
            ids = np.sort(rng.permutation(n_k)[:length])
            lists[h, r, :len(ids)] = ids
    lists[0, 0, 1:] = n_k                     # one valid id: all slices but one are empty
    lists[0, n_q - 1, :-1] = -1               # the last entry only
    lists[0, n_q - 1, -1] = n_k - 1
    lists[heads - 1, 0] = -1                  # none: zero rows
    return lists.astype(np.int32)


# 128 query blocks and, just past the rule, 132; last blocks of 1, 32, 33 and 64 rows; lists around each rule's edges, of
# fewer entries than slices, and (1 030) of more half tiles a slice than a pass of the decode holds
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("heads,frame_len,frames,length", [(2, 64, 4, 1), (2, 96, 4, 2), (2, 97, 4, 3), (32, 65, 5, 9), (33, 96, 5, 9),
                                                           (3, 31, 9, 8), (2, 97, 60, 65), (1, 64, 1030, 1030)])
def test_forward_of_few_query_blocks(gpu, heads, frame_len, frames, length, head_dim):  # noqa: F811
    torch, lf = gpu
    nb, f = -(-frame_len // 64), 2
    rng = np.random.default_rng(frame_len + length)
    mk = lambda t: synth.f32_to_bf16_bits(rng.standard_normal((heads, t * frame_len, head_dim), dtype=np.float32))
    x = {"Q": mk(f), "K": mk(frames), "V": mk(frames)}
    n_q, n_k = f * nb, frames * nb
    lists = _lists(rng, heads, n_q, n_k, length)
    print(f"few query blocks: {heads * n_q} d={head_dim} n={frame_len} list length {length}", flush=True)
    Q, K, V = (_dev(torch, x[k]) for k in "QKV")
    idx = torch.from_numpy(lists).cuda()
    out, lse2 = lf.lf_sparse_attn_fwd(Q, K, V, idx, frame_len, 64)
    again = lf.lf_sparse_attn(Q, K, V, idx, frame_len, 64)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), again.view(torch.int16))
    got, lse2 = out.float().cpu().numpy().astype(np.float64), lse2.cpu().numpy()
    Qf, Kf, Vf = (_host_f32(x[k]) for k in "QKV")
    for h, r in {(0, 0), (0, n_q - 1), (heads - 1, 0), (heads - 1, n_q - 1), (heads // 2, nb - 1)}:
        kept = [int(c) for c in lists[h, r] if 0 <= c < n_k]
        lo, hi = O.block_token_range(r, frame_len, 64)
        if not kept:
            assert not got[h, lo:hi].any() and np.isposinf(lse2[h, lo:hi]).all()
            continue
        err = np.abs(got[h, lo:hi] - O.sparse_attention_block(Qf[h], Kf[h], Vf[h], r, kept, frame_len, 64))
        assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS, (h, r, err.max(), err.mean())
        cols = np.concatenate([np.arange(*O.block_token_range(c, frame_len, 64)) for c in kept])
        s = Qf[h, lo:hi].astype(np.float64) @ Kf[h, cols].astype(np.float64).T / np.sqrt(head_dim) / np.log(2.0)
        top = s.max(axis=1)
        ref2 = top + np.log2(np.exp2(s - top[:, None]).sum(axis=1))
        # the row sum is of probabilities rounded to bfloat16: at most 2^-8 of it, 2^-8 / ln 2 in log2
        assert np.abs(lse2[h, lo:hi] - ref2).max() <= 2.0 ** -8 / np.log(2.0) + 1e-4


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("frame_len,keep", [(96, 2), (97, 7), (200, 19)])
def test_current_blocks_behind_the_read_entries(gpu, frame_len, keep, head_dim):  # noqa: F811
    """lf_sparse_attn_split on few query blocks, one pass: the list's first entries are read, the current chunk's blocks are
    taken without reading their entries."""
    torch, lf = gpu
    w = synth.small_ragged(frame_len=frame_len, chunk_idx=6, heads=2, head_dim=head_dim)
    x = synth.make_inputs(w)
    n_q, n_k = (t * w.blocks_per_frame for t in (w.frames_per_chunk, w.frames))
    b = lf.lf_chunk_budget(w.chunk_idx, w.schedule)
    b.n_sink = b.n_win = 0
    b.k_frames, b.k_blocks, b.list_len = w.hist_frames, keep, keep + n_q
    rng = np.random.default_rng(keep)
    lists = np.stack([np.stack([np.concatenate([np.sort(rng.permutation(n_k - n_q)[:keep]), np.arange(n_k - n_q, n_k)])
                                for _ in range(n_q)]) for _ in range(w.heads)]).astype(np.int32)
    Q, K, V = (_dev(torch, x[k]) for k in "QKV")
    unread = lists.copy()
    unread[:, :, keep:] = -7
    got = lf.lf_sparse_attn_split(Q, K, V, torch.from_numpy(unread).cuda(), frame_len, 64, b).float().cpu().numpy().astype(np.float64)
    Qf, Kf, Vf = (_host_f32(x[k]) for k in "QKV")
    for h in range(w.heads):
        for r in range(n_q):
            lo, hi = O.block_token_range(r, frame_len, 64)
            err = np.abs(got[h, lo:hi] - O.sparse_attention_block(Qf[h], Kf[h], Vf[h], r, [int(c) for c in lists[h, r]], frame_len, 64))
            assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS, (h, r, err.max(), err.mean())


def _gradients(torch, lf, rng, heads, frame_len, per_chunk, frames, head_dim, lists):
    mk = lambda t: synth.f32_to_bf16_bits(rng.standard_normal((heads, t * frame_len, head_dim), dtype=np.float32))
    x = {"Q": mk(per_chunk), "K": mk(frames), "V": mk(frames), "dO": mk(per_chunk)}
    Q, K, V, dO = (_dev(torch, x[k]) for k in ("Q", "K", "V", "dO"))
    idx = torch.from_numpy(lists).cuda()
    out, lse2 = lf.lf_sparse_attn_fwd(Q, K, V, idx, frame_len, 64)
    grads = tuple(torch.full_like(t, float("nan")) for t in (Q, K, V))
    runs = []
    for _ in range(2):
        lf.lf_sparse_attn_bwd(Q, K, V, out, dO, lse2, idx, frame_len, 64, grads=grads)
        torch.cuda.synchronize()
        runs.append([g.clone() for g in grads])
    assert all(torch.equal(a.view(torch.int16), b.view(torch.int16)) for a, b in zip(*runs))
    return x, [g.float().cpu().numpy().astype(np.float64) for g in runs[0]]


def _check_head(x, grads, lists, h, n_k, frame_len):
    """One head against the oracle; a query block without a valid id takes part with a zero upstream gradient."""
    Qf, Kf, Vf, dOf = (_host_f32(x[k])[h:h + 1].copy() for k in ("Q", "K", "V", "dO"))
    kept = np.empty((1, lists.shape[1]), dtype=object)
    for r in range(lists.shape[1]):
        kept[0, r] = [int(c) for c in lists[h, r] if 0 <= c < n_k]
        if not kept[0, r]:
            lo, hi = O.block_token_range(r, frame_len, 64)
            assert not grads[0][h, lo:hi].any()
            kept[0, r], dOf[0, lo:hi] = [0], 0
    for name, got, want in zip(("dQ", "dK", "dV"), grads, O.sparse_attention_backward(Qf, Kf, Vf, dOf, kept, frame_len, 64)):
        _close(name, got[h:h + 1], want)


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("heads,frame_len,frames,length", [(2, 64, 4, 3), (2, 96, 4, 4), (2, 97, 4, 5), (2, 65, 4, 6), (32, 65, 5, 9), (33, 96, 5, 9),
                                                           (3, 31, 9, 8), (1, 64, 1030, 1030)])
def test_dq_of_few_query_blocks(gpu, heads, frame_len, frames, length, head_dim):  # noqa: F811
    torch, lf = gpu
    nb = -(-frame_len // 64)
    rng = np.random.default_rng(frame_len + length)
    lists = _lists(rng, heads, 2 * nb, frames * nb, length)
    print(f"few query blocks, backward: {heads * 2 * nb} d={head_dim} n={frame_len} list length {length}", flush=True)
    x, grads = _gradients(torch, lf, rng, heads, frame_len, 2, frames, head_dim, lists)
    for h in {0, heads - 1}:
        _check_head(x, grads, lists, h, frames * nb, frame_len)


# 128 and 132 KV blocks (the edge at d = 128), 352 and 360 (at d = 64); last blocks of 1, 32, 33 and 64 rows; transposed lists of 0, 1, odd
# and even lengths and of every query block
@pytest.mark.parametrize("head_dim,heads,frame_len,per_chunk,frames,length", [
    (128, 32, 65, 2, 2, 3), (128, 33, 96, 2, 2, 3), (64, 44, 97, 2, 4, 5), (64, 45, 97, 2, 4, 5), (128, 2, 96, 3, 9, 1), (64, 2, 31, 3, 9, 2),
    (128, 1, 64, 5, 20, 11), (64, 1, 65, 5, 20, 11), (128, 1, 64, 128, 128, 128), (64, 1, 64, 352, 352, 40)])
def test_gradients_of_few_kv_blocks(gpu, head_dim, heads, frame_len, per_chunk, frames, length):  # noqa: F811
    torch, lf = gpu
    nb = -(-frame_len // 64)
    rng = np.random.default_rng(frame_len + length)
    lists = _lists(rng, heads, per_chunk * nb, frames * nb, length)
    first = lists[:, 1:, 0]
    first[(first >= 0) & (first < frames * nb)] = 0                       # KV block 0 is in (nearly) every list
    print(f"few KV blocks: {heads * frames * nb} d={head_dim} n={frame_len} list length {length}", flush=True)
    x, grads = _gradients(torch, lf, rng, heads, frame_len, per_chunk, frames, head_dim, lists)
    for h in {0, heads - 1}:
        _check_head(x, grads, lists, h, frames * nb, frame_len)


# Lists in two parts: 132, 256, 258, 512, 516 (and at d = 64 768, 772) query blocks, list lengths at both ends of the rules
@pytest.mark.parametrize("head_dim,heads,frame_len,length", [
    (128, 33, 97, 2), (128, 33, 96, 14), (128, 64, 65, 15), (128, 129, 64, 8), (128, 128, 97, 9), (128, 129, 97, 9), (128, 128, 96, 129),
    (64, 33, 97, 3), (64, 64, 96, 10), (64, 64, 65, 11), (64, 129, 64, 6), (64, 129, 97, 7), (64, 192, 96, 9), (64, 193, 65, 9), (64, 129, 64, 140)])
def test_lists_in_two_parts(gpu, head_dim, heads, frame_len, length):  # noqa: F811
    torch, lf = gpu
    nb = -(-frame_len // 64)
    frames = max(2, -(-length // nb) + 1)
    rng = np.random.default_rng(frame_len + length)
    n_q, n_k = 2 * nb, frames * nb
    lists = _lists(rng, heads, n_q, n_k, length)
    print(f"two parts: {heads * n_q} blocks d={head_dim} n={frame_len} list length {length}", flush=True)
    x, grads = _gradients(torch, lf, rng, heads, frame_len, 2, frames, head_dim, lists)
    Q, K, V = (_dev(torch, x[k]) for k in "QKV")
    got = lf.lf_sparse_attn(Q, K, V, torch.from_numpy(lists).cuda(), frame_len, 64).float().cpu().numpy().astype(np.float64)
    for h in {0, heads - 1}:
        _check_head(x, grads, lists, h, n_k, frame_len)
        Qf, Kf, Vf = (_host_f32(x[k][h]) for k in "QKV")
        for r in range(n_q):
            kept = [int(c) for c in lists[h, r] if 0 <= c < n_k]
            lo, hi = O.block_token_range(r, frame_len, 64)
            ref = O.sparse_attention_block(Qf, Kf, Vf, r, kept, frame_len, 64) if kept else 0.0
            err = np.abs(got[h, lo:hi] - ref)
            assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS, (h, r, err.max(), err.mean())
