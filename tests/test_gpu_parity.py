"""Parity of the HIP path (through the C ABI) with the CPU oracle on the same seeded inputs.

Bars: index lists, pooled block/frame means -- bit-exact; attention output -- max-abs 2e-2 and
mean-abs 2e-3 against the binary64 oracle (bf16 inputs, bf16 output)."""
import numpy as np
import pytest

from oracle import hsa_oracle as O
from paper_2602_04789_amd import synth

pytestmark = pytest.mark.gpu

MAX_ABS, MEAN_ABS = 2e-2, 2e-3


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_04789_amd import lf
    lf.load()
    return torch, lf


def _dev(torch, bits):
    return torch.from_numpy(bits).view(torch.bfloat16).cuda()


def _host_f32(bits):
    return synth.bf16_bits_to_f32(bits)


def _run_select(torch, lf, w, x, check_intermediates=True):
    """GPU lists vs oracle lists (all heads, all query blocks); returns (gpu tensors, lists)."""
    Q, K, V = (_dev(torch, x[k]) for k in "QKV")
    b = lf.lf_chunk_budget(w.chunk_idx, w.schedule)
    ob = O.chunk_budget(w.chunk_idx, w.schedule)
    assert b.list_len == ob.list_len and b.k_blocks == ob.k_blocks
    sh = lf.make_shape(Q, K, frame_len=w.frame_len, block=w.block)
    ws = torch.empty(lf.lf_workspace_bytes(sh, b), dtype=torch.uint8, device="cuda")
    idx = lf.lf_select_mask(Q, K, w.frame_len, w.block, b, workspace=ws)
    torch.cuda.synchronize()
    want, I = O.select_mask(_host_f32(x["Q"]), _host_f32(x["K"]), w.frame_len, w.block, ob,
                            return_intermediates=True)
    if check_intermediates:
        off = lf.lf_workspace_layout(sh, b)
        H, d = w.heads, w.head_dim
        raw = ws.cpu().numpy()
        for name, o, cnt in (("q_tilde", off[0], I["q_tilde"].shape[1]),
                             ("k_tilde", off[1], I["k_tilde"].shape[1]),
                             ("k_hat", off[2], I["k_hat"].shape[1] if ob.k_frames < len(I["M"]) else 0)):
            if cnt == 0:
                continue
            got = raw[o:o + H * cnt * d * 4].view(np.float32)
            if name == "q_tilde":
                got = got.reshape(H, cnt, d)
            else:   # channel-quad major: [H][d/4][rows][4]
                got = got.reshape(H, d // 4, cnt, 4).transpose(0, 2, 1, 3).reshape(H, cnt, d)
            got = np.ascontiguousarray(got)
            assert np.array_equal(got.view(np.uint32), I[name].view(np.uint32)), name
    got = idx.cpu().numpy()
    assert got.shape == want.shape and got.dtype == np.int32
    bad = np.argwhere((got != want).any(axis=-1))
    assert bad.size == 0, f"{len(bad)} of {got.shape[0] * got.shape[1]} lists differ, first {bad[:3]}"
    return (Q, K, V), idx, want


def _check_attn(torch, lf, w, x, dev, idx, lists, pairs=None, split=False):
    """lf_sparse_attn (or, with split, lf_sparse_attn_split) against the oracle's Eq. 13."""
    Q, K, V = dev
    if split:
        b = lf.lf_chunk_budget(w.chunk_idx, w.schedule)
        out = lf.lf_sparse_attn_split(Q, K, V, idx, w.frame_len, w.block, b)
    else:
        out = lf.lf_sparse_attn(Q, K, V, idx, w.frame_len, w.block)
    torch.cuda.synchronize()
    got = out.float().cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all()
    Qf, Kf, Vf = (_host_f32(x[k]) for k in "QKV")
    nb = w.blocks_per_frame
    n_q = w.frames_per_chunk * nb
    if pairs is None:
        pairs = [(h, r) for h in range(w.heads) for r in range(n_q)]
    worst, total, count = 0.0, 0.0, 0
    for h, r in pairs:
        lo, hi = O.block_token_range(r, w.frame_len, w.block)
        ref = O.sparse_attention_block(Qf[h], Kf[h], Vf[h], r, lists[h, r], w.frame_len, w.block)
        err = np.abs(got[h, lo:hi] - ref)
        worst = max(worst, float(err.max()))
        total += float(err.sum())
        count += err.size
    mean = total / count
    assert worst <= MAX_ABS and mean <= MEAN_ABS, (worst, mean)
    return got, worst, mean


def _sample_pairs(w, k, seed=0):
    rng = np.random.default_rng(seed)
    nb = w.blocks_per_frame
    n_q = w.frames_per_chunk * nb
    pairs = {(0, 0), (w.heads - 1, n_q - 1), (w.heads // 2, nb - 1)}   # includes ragged query blocks
    while len(pairs) < k:
        pairs.add((int(rng.integers(w.heads)), int(rng.integers(n_q))))
    return sorted(pairs)


# ----------------------------------------------------------------------------- small cases, all outputs

SMALL = {
    "tiny": lambda: synth.cfg_tiny(),
    "ragged_c1": lambda: synth.small_ragged(chunk_idx=1, current_mandatory=0),
    "ragged_c2": lambda: synth.small_ragged(chunk_idx=2),
    "ragged_c4": lambda: synth.small_ragged(chunk_idx=4),
    "ragged_c6_d64": lambda: synth.small_ragged(chunk_idx=6, head_dim=64, heads=2),
    "ragged_compete": lambda: synth.small_ragged(chunk_idx=4, current_mandatory=0,
                                                 ratio_of=synth.OF_ALL, keep_fixed=0.3),
    "aligned_1536_c3": lambda: synth.scaled(synth.cfg_paper_5s(3, heads=2)),
    "one_token_tail": lambda: synth.small_ragged(frame_len=129, chunk_idx=3, heads=2),
    "short_frame": lambda: synth.small_ragged(frame_len=40, chunk_idx=5, heads=2, k_frames=1),
    # last block of 31, 32 and 33 tokens: around the 32-row half tiles of the attention kernel
    "tail_31": lambda: synth.small_ragged(frame_len=95, chunk_idx=3, heads=2),
    "tail_32": lambda: synth.small_ragged(frame_len=96, chunk_idx=3, heads=2),
    "tail_33": lambda: synth.small_ragged(frame_len=97, chunk_idx=3, heads=2, head_dim=64),
    "many_frames": lambda: synth.small_ragged(frame_len=64, chunk_idx=40, frames_per_chunk=2,
                                              heads=1, k_frames=5, n_sink=2, n_win=3),
    # 216 candidates of which 200 are known before the frame ranking (10 sink + 10 window frames and
    # 5 competing current frames of 8 blocks): the early scoring reaches down into the wavefront
    # that also scores the frames and the retrieved blocks
    "known_200_of_216": lambda: synth.small_ragged(frame_len=500, chunk_idx=6, frames_per_chunk=5, heads=1,
                                                   k_frames=2, n_sink=10, n_win=10, current_mandatory=0,
                                                   ratio_of=synth.OF_CANDIDATES, keep_fixed=0.5),
    # candidate sets wider than one per thread: 320, 560 and 1040 candidate blocks
    "wide_320": lambda: synth.small_ragged(frame_len=500, chunk_idx=28, frames_per_chunk=5, heads=1,
                                           k_frames=35, n_sink=2, n_win=3,
                                           ratio_of=synth.OF_CANDIDATES, keep_fixed=0.5),
    "wide_560": lambda: synth.small_ragged(frame_len=500, chunk_idx=28, frames_per_chunk=5, heads=1,
                                           k_frames=65, n_sink=2, n_win=3,
                                           ratio_of=synth.OF_CANDIDATES, keep_fixed=0.3),
    "wide_1040_compete": lambda: synth.small_ragged(frame_len=500, chunk_idx=28, frames_per_chunk=5,
                                                    heads=1, k_frames=120, n_sink=2, n_win=3,
                                                    current_mandatory=0,
                                                    ratio_of=synth.OF_CANDIDATES, keep_fixed=0.1),
}


@pytest.mark.parametrize("name", list(SMALL))
def test_small_cases_match_oracle_everywhere(gpu, name):
    torch, lf = gpu
    w = SMALL[name]()
    x = synth.make_inputs(w)
    print(f"case {name}: H={w.heads} d={w.head_dim} n={w.frame_len} F={w.frames}", flush=True)
    dev, idx, lists = _run_select(torch, lf, w, x)
    _check_attn(torch, lf, w, x, dev, idx, lists)
    _check_attn(torch, lf, w, x, dev, idx, lists, split=True)


def test_ties_resolve_to_lower_index(gpu):
    """Duplicate history frames and duplicate blocks: equal float32 scores everywhere."""
    torch, lf = gpu
    w = synth.small_ragged(chunk_idx=5, heads=2, k_frames=2, keep_fixed=0.3)
    x = synth.make_inputs(w)
    n = w.frame_len
    K = x["K"]
    K[:, 3 * n:4 * n] = K[:, 2 * n:3 * n]          # frame 3 := frame 2
    K[:, 4 * n:5 * n] = K[:, 2 * n:3 * n]          # frame 4 := frame 2
    K[:, 2 * n + 64:2 * n + 128] = K[:, 2 * n:2 * n + 64]   # block 1 := block 0 inside frame 2
    K[:, n:2 * n] = 0                               # an all-zero frame: scores of +0.0 / -0.0
    dev, idx, lists = _run_select(torch, lf, w, x)
    _check_attn(torch, lf, w, x, dev, idx, lists)


def test_full_budget_equals_dense_attention(gpu):
    torch, lf = gpu
    w = synth.small_ragged(chunk_idx=3, heads=2)
    x = synth.make_inputs(w)
    Q, K, V = (_dev(torch, x[k]) for k in "QKV")
    lists = O.full_lists(w.heads, w.frame_len, w.block, w.frames_per_chunk, w.frames)
    idx = torch.from_numpy(lists).cuda()
    out = lf.lf_sparse_attn(Q, K, V, idx, w.frame_len, w.block)
    ref = torch.nn.functional.scaled_dot_product_attention(Q.float(), K.float(), V.float())
    torch.cuda.synchronize()
    err = (out.float() - ref).abs()
    assert err.max().item() <= MAX_ABS and err.mean().item() <= MEAN_ABS


def test_attention_list_edge_cases(gpu):
    """Single tail block; unordered list; out-of-range ids skipped; duplicate id counted twice;
    head-strided (non-contiguous) tensors; explicit softmax scale."""
    torch, lf = gpu
    w = synth.small_ragged(chunk_idx=3, heads=2)
    x = synth.make_inputs(w)
    Qf, Kf, Vf = (_host_f32(x[k]) for k in "QKV")
    nb, n_q, n_k = w.blocks_per_frame, w.frames_per_chunk * w.blocks_per_frame, w.frames * w.blocks_per_frame
    # tensors carved out of a larger buffer: head stride != q_len * d, token stride != d
    def strided(bits):
        H, L, d = bits.shape
        buf = torch.zeros((H, L + 5, d + 8), dtype=torch.bfloat16, device="cuda")
        view = buf[:, 2:2 + L, :d]
        view.copy_(_dev(torch, bits))
        return view
    Q, K, V = strided(x["Q"]), strided(x["K"]), strided(x["V"])
    Obuf = torch.zeros((w.heads, w.q_len + 3, w.head_dim + 8), dtype=torch.bfloat16, device="cuda")
    Oview = Obuf[:, 1:1 + w.q_len, :w.head_dim]

    cases = {
        "single_tail_block": np.full((w.heads, n_q, 1), nb - 1, np.int32),
        "unordered": np.tile(np.array([n_k - 1, 0, 5, 2], np.int32), (w.heads, n_q, 1)),
        "invalid_ids_skipped": np.tile(np.array([-1, 3, n_k, 1 << 30, 4], np.int32), (w.heads, n_q, 1)),
        "duplicate": np.tile(np.array([2, 2, 7], np.int32), (w.heads, n_q, 1)),
        # long lists.  With these few query blocks they are divided among four pairs of wavefronts, which
        # decode 128 entries of their quarter per pass; the edges of the passes of either form are in
        # test_list_lengths_around_the_decode_passes
        "len_255": np.tile((np.arange(255, dtype=np.int32) * 5) % n_k, (w.heads, n_q, 1)),
        "len_256": np.tile((np.arange(256, dtype=np.int32) * 5) % n_k, (w.heads, n_q, 1)),
        "len_257": np.tile((np.arange(257, dtype=np.int32) * 5) % n_k, (w.heads, n_q, 1)),
        "len_513": np.tile((np.arange(513, dtype=np.int32) * 3) % n_k, (w.heads, n_q, 1)),
        "len_1100": np.tile((np.arange(1100, dtype=np.int32) * 7) % n_k, (w.heads, n_q, 1)),
    }
    # a query block whose list holds no valid id at all gives zero rows (stated in the header)
    some_invalid = np.tile(np.array([3, 1, 4], np.int32), (w.heads, n_q, 1))
    some_invalid[0, 1] = (-1, n_k, 1 << 30)
    some_invalid[1, n_q - 1] = (-5, -1, n_k + 7)
    cases["a_list_without_valid_ids"] = some_invalid
    for name, lists in cases.items():
        print("edge case", name, flush=True)
        idx = torch.from_numpy(lists).cuda()
        scale = 0.05 if name == "unordered" else 0.0
        out = lf.lf_sparse_attn(Q, K, V, idx, w.frame_len, w.block, softmax_scale=scale, O=Oview)
        torch.cuda.synchronize()
        got = out.float().cpu().numpy().astype(np.float64)
        for h in range(w.heads):
            for r in range(n_q):
                kept = [int(c) for c in lists[h, r] if 0 <= c < n_k]
                lo, hi = O.block_token_range(r, w.frame_len, w.block)
                if not kept:
                    assert np.all(got[h, lo:hi] == 0.0), (name, h, r)
                    continue
                ref = O.sparse_attention_block(Qf[h], Kf[h], Vf[h], r, kept, w.frame_len, w.block,
                                               scale=(scale if scale else None))
                err = np.abs(got[h, lo:hi] - ref)
                assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS, (name, h, r, err.max())
    # nothing outside the O view was touched
    assert float(Obuf[:, 0].abs().max()) == 0 and float(Obuf[:, :, w.head_dim:].abs().max()) == 0


@pytest.mark.parametrize("frame_len,head_dim", [(200, 128), (232, 128), (224, 64)])
def test_lists_whose_half_tile_counts_differ(gpu, frame_len, head_dim):
    """A listed block of at most 32 tokens is one step of the kernel, a longer one two, an id out
    of range none, and the query blocks of a workgroup (in a call of so few: the four parts of a
    divided list) take the longest one's step count: lists of equal length whose neighbours differ in all of that (only tail blocks, only full blocks, a
    mix with invalid ids, hardly any valid id), with tails of 8, 40 and 32 tokens, two query
    frames so that a short query block sits inside the chunk, and more than one decode pass."""
    torch, lf = gpu
    w = synth.small_ragged(frame_len=frame_len, chunk_idx=4, heads=2, head_dim=head_dim)
    x = synth.make_inputs(w)
    Qf, Kf, Vf = (_host_f32(x[k]) for k in "QKV")
    Q, K, V = (_dev(torch, x[k]) for k in "QKV")
    nb, n_q, n_k = w.blocks_per_frame, w.frames_per_chunk * w.blocks_per_frame, w.frames * w.blocks_per_frame
    tails = np.arange(nb - 1, n_k, nb, dtype=np.int32)
    full = np.array([c for c in range(n_k) if c % nb != nb - 1], np.int32)
    rng = np.random.default_rng(7)
    for L in (6, 300):
        lists = np.empty((w.heads, n_q, L), np.int32)
        for h in range(w.heads):
            for r in range(n_q):
                kind = (r + h) % 4
                if kind == 0:
                    row = rng.choice(tails, L)
                elif kind == 1:
                    row = rng.choice(full, L)
                elif kind == 2:
                    row = rng.integers(-3, n_k + 3, L).astype(np.int32)
                else:
                    row = np.full(L, -1, np.int32)
                    row[rng.integers(0, L)] = rng.integers(0, n_k)
                lists[h, r] = row
        print(f"half-tile counts: n={frame_len} d={head_dim} list length {L}", flush=True)
        out = lf.lf_sparse_attn(Q, K, V, torch.from_numpy(lists).cuda(), w.frame_len, w.block)
        torch.cuda.synchronize()
        got = out.float().cpu().numpy().astype(np.float64)
        for h in range(w.heads):
            for r in range(n_q):
                kept = [int(c) for c in lists[h, r] if 0 <= c < n_k]
                lo, hi = O.block_token_range(r, w.frame_len, w.block)
                ref = O.sparse_attention_block(Qf[h], Kf[h], Vf[h], r, kept, w.frame_len, w.block)
                err = np.abs(got[h, lo:hi] - ref)
                assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS, (L, h, r, err.max())


@pytest.mark.parametrize("scale", [0.25, 1.0, 4.0])
def test_attention_with_extreme_logits(gpu, scale):
    """Logits far outside the usual range (softmax_scale 0.25, 1 and 4 instead of 1/sqrt(d) =
    0.088: tens to hundreds in the exp2 domain, rising and falling from tile to tile, beyond what
    exp2 holds in float32): the reference of the online softmax has to move, nothing may
    overflow, and the usual tolerance still holds (the scale is applied to the float32 scores,
    not folded into a bfloat16 operand)."""
    torch, lf = gpu
    w = synth.small_ragged(chunk_idx=4, heads=2)
    x = synth.make_inputs(w)
    n = w.frame_len
    K = x["K"].copy()
    Kf = _host_f32(K)
    Kf[:, 0:n] *= 0.05          # a first frame with tiny logits, then much larger ones
    Kf[:, 2 * n:3 * n] *= 3.0
    K = synth.f32_to_bf16_bits(Kf)
    Q, Kd, V = _dev(torch, x["Q"]), _dev(torch, K), _dev(torch, x["V"])
    lists = O.full_lists(w.heads, w.frame_len, w.block, w.frames_per_chunk, w.frames)
    idx = torch.from_numpy(lists).cuda()
    out = lf.lf_sparse_attn(Q, Kd, V, idx, w.frame_len, w.block, softmax_scale=scale)
    torch.cuda.synchronize()
    got = out.float().cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all()
    Qf, Kf, Vf = _host_f32(x["Q"]), _host_f32(K), _host_f32(x["V"])
    n_q = lists.shape[1]
    worst = 0.0
    for h in range(w.heads):
        for r in range(0, n_q, 3):
            lo, hi = O.block_token_range(r, w.frame_len, w.block)
            ref = O.sparse_attention_block(Qf[h], Kf[h], Vf[h], r, list(lists[h, r]), w.frame_len,
                                           w.block, scale=scale)
            err = np.abs(got[h, lo:hi] - ref)
            worst = max(worst, float(err.max()))
            assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS, (h, r, err.max(), err.mean())
    print(f"extreme logits, scale {scale}: max-abs {worst:.2e}", flush=True)


def test_pooled_key_cache_gives_the_same_lists(gpu):
    """A rollout with the pooled-key cache: history frames are pooled once, when their chunk is
    current; every call pools only Q and the current chunk.  Lists must equal those of the
    stateless call (and so the oracle's) bit for bit, also after the current chunk's keys change
    between two steps of the same chunk."""
    torch, lf = gpu
    last = synth.small_ragged(chunk_idx=5, heads=3)
    xk = synth.make_inputs(last)
    n, f, max_frames = last.frame_len, last.frames_per_chunk, last.frames + 2
    Kall = _dev(torch, xk["K"])
    sh_full = lf.make_shape(Kall[:, :f * n], Kall, frame_len=n, block=last.block)
    kc = torch.zeros(lf.lf_kcache_bytes(sh_full, max_frames), dtype=torch.uint8, device="cuda")
    for chunk in range(1, 6):
        w = synth.small_ragged(chunk_idx=chunk, heads=3)
        x = synth.make_inputs(w)
        Q = _dev(torch, x["Q"])
        K = Kall[:, :w.frames * n].clone()
        b = lf.lf_chunk_budget(chunk, w.schedule)
        for step in range(2):
            if step == 1:   # the chunk being denoised changes between steps
                K[:, w.hist_frames * n:] = _dev(torch, x["K"])[:, w.hist_frames * n:]
            if step == 0:   # two ways to bring the current chunk in: a separate update ...
                lf.lf_kcache_update(K, n, w.block, w.hist_frames, w.frames, max_frames, kc)
                got = lf.lf_select_mask_cached(Q, kc, max_frames, w.frames * n, n, w.block, b)
            else:           # ... or together with the selection
                got = lf.lf_select_mask_cached(Q, kc, max_frames, w.frames * n, n, w.block, b, Kcache=K)
            want = lf.lf_select_mask(Q, K, n, w.block, b)
            torch.cuda.synchronize()
            assert torch.equal(got, want), (chunk, step)
            # ... and the oracle's, at every step of every chunk
            Kf = K.view(torch.int16).cpu().numpy().view(np.uint16)
            ob = O.chunk_budget(chunk, w.schedule)
            ref = O.select_mask(_host_f32(x["Q"]), _host_f32(Kf), n, w.block, ob)
            assert np.array_equal(got.cpu().numpy(), ref), (chunk, step)
        # commit the chunk: its final keys are the ones of the shared history
        lf.lf_kcache_update(Kall[:, :w.frames * n], n, w.block, w.hist_frames, w.frames, max_frames, kc)
    with pytest.raises(lf.LfError):
        lf.lf_kcache_update(Kall, n, last.block, 0, last.frames + 1, max_frames, kc)


def test_calls_are_deterministic(gpu):
    torch, lf = gpu
    w = synth.small_ragged(chunk_idx=4)
    x = synth.make_inputs(w)
    Q, K, V = (_dev(torch, x[k]) for k in "QKV")
    b = lf.lf_chunk_budget(w.chunk_idx, w.schedule)
    i1 = lf.lf_select_mask(Q, K, w.frame_len, w.block, b)
    o1 = lf.lf_sparse_attn(Q, K, V, i1, w.frame_len, w.block)
    i2 = lf.lf_select_mask(Q, K, w.frame_len, w.block, b)
    o2 = lf.lf_sparse_attn(Q, K, V, i2, w.frame_len, w.block)
    torch.cuda.synchronize()
    assert torch.equal(i1, i2) and torch.equal(o1.view(torch.int16), o2.view(torch.int16))


@pytest.mark.parametrize("frame_len,head_dim", [(129, 128), (400, 128), (200, 64)])
def test_nothing_is_read_or_written_outside_the_tensors(gpu, frame_len, head_dim):
    """The last block of a frame is short, and the last frame ends the cache.  Every tensor is
    placed in a buffer whose surroundings hold NaN: a read past a short block or past the end of
    the cache would poison the output (0 * NaN), a write outside O would change a guard."""
    torch, lf = gpu
    w = synth.small_ragged(frame_len=frame_len, chunk_idx=3, heads=2, head_dim=head_dim)
    x = synth.make_inputs(w)
    plain = [_dev(torch, x[k]) for k in "QKV"]
    b = lf.lf_chunk_budget(w.chunk_idx, w.schedule)
    idx0 = lf.lf_select_mask(plain[0], plain[1], w.frame_len, w.block, b)
    out0 = lf.lf_sparse_attn(*plain, idx0, w.frame_len, w.block)
    pad = 64 * head_dim * 2   # one full tile of elements before and after

    def guarded(t):
        buf = torch.full((t.numel() + 2 * pad,), float("nan"), dtype=torch.bfloat16, device="cuda")
        view = buf[pad:pad + t.numel()].view(t.shape)
        view.copy_(t)
        return buf, view

    (_, Q), (_, K), (_, V) = (guarded(t) for t in plain)
    obuf, Oview = guarded(torch.zeros_like(plain[0]))
    idx = lf.lf_select_mask(Q, K, w.frame_len, w.block, b)
    lf.lf_sparse_attn(Q, K, V, idx, w.frame_len, w.block, O=Oview)
    torch.cuda.synchronize()
    assert torch.equal(idx, idx0)
    assert torch.isfinite(Oview.float()).all()
    assert torch.equal(Oview.view(torch.int16), out0.view(torch.int16))
    assert torch.isnan(obuf[:pad].float()).all() and torch.isnan(obuf[pad + Oview.numel():].float()).all()


def test_step_replays_from_a_captured_graph(gpu):
    """Selection + attention captured once into a HIP graph (no allocation, memset or
    synchronisation inside the library) and replayed on new inputs written into the same
    buffers, with eager work and synchronisations between the replays; every replay must
    equal the eager result bit for bit."""
    torch, lf = gpu
    w = synth.small_ragged(chunk_idx=4)
    b = lf.lf_chunk_budget(w.chunk_idx, w.schedule)
    xs = [synth.make_inputs(synth.small_ragged(chunk_idx=4, seed=s)) for s in (11, 12, 13)]
    Q, K, V = (_dev(torch, xs[0][k]).clone() for k in "QKV")
    sh = lf.make_shape(Q, K, frame_len=w.frame_len, block=w.block)
    ws = torch.empty(lf.lf_workspace_bytes(sh, b), dtype=torch.uint8, device="cuda")
    nq = w.frames_per_chunk * w.blocks_per_frame
    idx = torch.empty((w.heads, nq, b.list_len), dtype=torch.int32, device="cuda")
    out = torch.empty_like(Q)

    def step():
        lf.lf_select_mask(Q, K, w.frame_len, w.block, b, indices=idx, workspace=ws)
        lf.lf_sparse_attn(Q, K, V, idx, w.frame_len, w.block, O=out)

    step()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step()
    for x in xs[1:] + xs[:1] + xs[1:2]:
        for t, k in ((Q, "Q"), (K, "K"), (V, "V")):
            t.copy_(_dev(torch, x[k]))
        idx.fill_(-7)
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        got_idx, got_out = idx.clone(), out.clone()
        want_idx = lf.lf_select_mask(Q, K, w.frame_len, w.block, b)
        want_out = lf.lf_sparse_attn(Q, K, V, want_idx, w.frame_len, w.block)
        torch.cuda.synchronize()
        assert torch.equal(got_idx, want_idx)
        assert torch.equal(got_out.view(torch.int16), want_out.view(torch.int16))


def test_binding_rejects_bad_arguments(gpu):
    torch, lf = gpu
    w = synth.cfg_tiny()
    x = synth.make_inputs(w)
    Q, K, V = (_dev(torch, x[k]) for k in "QKV")
    b = lf.lf_chunk_budget(w.chunk_idx, w.schedule)
    with pytest.raises(lf.LfError):
        lf.lf_select_mask(Q, K, w.frame_len + 1, w.block, b)
    with pytest.raises(lf.LfError):
        lf.lf_select_mask(Q, K, w.frame_len, w.block, b,
                          workspace=torch.empty(256, dtype=torch.uint8, device="cuda"))
    with pytest.raises(ValueError):
        lf.lf_select_mask(Q.float(), K, w.frame_len, w.block, b)
    with pytest.raises(ValueError):
        lf.lf_sparse_attn(Q, K, V, torch.zeros((1, 1, 1), dtype=torch.int32, device="cuda"),
                          w.frame_len, w.block)


# ----------------------------------------------------------------------------- full-size configurations

FULL = {
    "first_chunk": synth.cfg_first_chunk,
    "mid_rollout": synth.cfg_mid_rollout,
    "last_chunk": synth.cfg_last_chunk,
    # the paper's own operating point (Experimental Details; hyper-parameter table)
    "paper5s_mid": lambda: synth.cfg_paper_5s(4),
    "paper5s_last": lambda: synth.cfg_paper_5s(7),
    "paper15s_late": lambda: synth.cfg_paper_15s(20),   # 57 history frames, 54 of them candidates
}


@pytest.mark.parametrize("name", list(FULL))
def test_full_size_configs(gpu, name):
    """Benchmark shapes in the launch configuration the benchmark times: every index list and
    every (head, query block) of the attention output against the oracle."""
    torch, lf = gpu
    w = FULL[name]()
    print(f"config {name}: generating", flush=True)
    x = synth.make_inputs(w)
    print("select parity", flush=True)
    dev, idx, lists = _run_select(torch, lf, w, x)
    print("attention parity (all query blocks)", flush=True)
    got, worst, mean = _check_attn(torch, lf, w, x, dev, idx, lists)
    print(f"{name}: max-abs {worst:.2e} mean-abs {mean:.2e}", flush=True)
    if w.schedule.current_mandatory and w.hist_frames > 0:
        print("attention parity, dense + list-driven phases (all query blocks)", flush=True)
        _, worst2, mean2 = _check_attn(torch, lf, w, x, dev, idx, lists, split=True)
        print(f"{name} split: max-abs {worst2:.2e} mean-abs {mean2:.2e}", flush=True)
    # size-independent properties on the whole output: finite; |O| bounded by max |V|
    vmax = float(np.abs(_host_f32(x["V"])).max())
    assert np.abs(got).max() <= vmax * 1.01


@pytest.mark.parametrize("step", [0, 3])
@pytest.mark.parametrize("chunk", [1, 2, 3, 4, 5, 6, 7])
def test_rollout_calls_40_heads(gpu, chunk, step):
    """The 40-head rollout: all seven chunks at the first and the last denoising step.  Every
    index list of all 40 heads against the oracle; the attention output of every query block of
    three heads (the oracle would need minutes for all 40)."""
    torch, lf = gpu
    w = synth.cfg_rollout(chunk, step=step)
    print(f"rollout chunk {chunk} step {step}: generating", flush=True)
    x = synth.make_inputs(w)
    print("select parity", flush=True)
    dev, idx, lists = _run_select(torch, lf, w, x, check_intermediates=False)
    print("attention parity (heads 0, 19, 39)", flush=True)
    n_q = w.frames_per_chunk * w.blocks_per_frame
    pairs = [(h, r) for h in (0, 19, 39) for r in range(n_q)]
    _, worst, mean = _check_attn(torch, lf, w, x, dev, idx, lists, pairs=pairs)
    print(f"rollout chunk {chunk} step {step}: max-abs {worst:.2e} mean-abs {mean:.2e}", flush=True)
    _, worst, mean = _check_attn(torch, lf, w, x, dev, idx, lists, pairs=pairs, split=True)
    print(f"rollout chunk {chunk} step {step} split: max-abs {worst:.2e} mean-abs {mean:.2e}", flush=True)


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("heads,list_len", [(2, 5), (2, 6), (2, 7), (8, 31), (16, 31), (16, 32), (16, 33), (17, 32),
                                            (16, 95), (16, 96), (17, 96), (2, 129), (2, 517)])
def test_lists_divided_among_the_wavefronts_of_a_workgroup(gpu, heads, list_len, head_dim):
    """The attention kernels divide lists among four pairs of wavefronts when a call has few query
    blocks: both sides of each edge of that rule (list lengths 5/6, for more than 256 query blocks 31/32 at
    d = 64 and 95/96 at d = 128; 512 and 544 query blocks), slices of unequal length, slices without any valid id, several decode passes, ragged
    query blocks, a continued state (the two-phase call) and the log-sum-exp, on lists with
    out-of-range and repeated ids."""
    torch, lf = gpu
    w = synth.small_ragged(frame_len=1000, chunk_idx=2, heads=heads, head_dim=head_dim)
    x = synth.make_inputs(w)
    Qf, Kf, Vf = (_host_f32(x[k]) for k in "QKV")
    Q, K, V = (_dev(torch, x[k]) for k in "QKV")
    n_q, n_k = w.frames_per_chunk * w.blocks_per_frame, w.frames * w.blocks_per_frame
    rng = np.random.default_rng(list_len)
    lists = rng.integers(-2, n_k + 2, (heads, n_q, list_len)).astype(np.int32)
    lists[0, 0, 1:] = -1                                  # one valid id: three empty slices
    lists[0, 0, 0] = 3
    lists[heads - 1, n_q - 1, :list_len // 2] = n_k       # the first slices empty, and a ragged query block
    lists[heads - 1, n_q - 1, list_len - 1] = 0
    lists[heads - 1, 0] = -1                              # none: zero rows
    print(f"divided lists: heads={heads} d={head_dim} list length {list_len}", flush=True)
    idx = torch.from_numpy(lists).cuda()
    out, lse2 = lf.lf_sparse_attn_fwd(Q, K, V, idx, w.frame_len, w.block)
    assert torch.equal(out, lf.lf_sparse_attn(Q, K, V, idx, w.frame_len, w.block))
    torch.cuda.synchronize()
    got, lse2 = out.float().cpu().numpy().astype(np.float64), lse2.cpu().numpy()
    pairs = {(0, 0), (heads - 1, n_q - 1), (heads - 1, 0), (0, w.blocks_per_frame - 1)}
    while len(pairs) < 24:
        pairs.add((int(rng.integers(heads)), int(rng.integers(n_q))))
    for h, r in sorted(pairs):
        kept = [int(c) for c in lists[h, r] if 0 <= c < n_k]
        lo, hi = O.block_token_range(r, w.frame_len, w.block)
        if not kept:
            assert np.all(got[h, lo:hi] == 0.0) and np.isposinf(lse2[h, lo:hi]).all()
            continue
        ref = O.sparse_attention_block(Qf[h], Kf[h], Vf[h], r, kept, w.frame_len, w.block)
        err = np.abs(got[h, lo:hi] - ref)
        assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS, (h, r, err.max())
        cols = np.concatenate([np.arange(*O.block_token_range(c, w.frame_len, w.block)) for c in kept])
        s = Qf[h, lo:hi].astype(np.float64) @ Kf[h, cols].astype(np.float64).T / np.sqrt(head_dim) / np.log(2.0)
        top = s.max(axis=1)
        ref2 = top + np.log2(np.exp2(s - top[:, None]).sum(axis=1))
        # the row sum is of probabilities rounded to bfloat16: at most 2^-8 of it, 2^-8 / ln 2 in log2
        assert np.abs(lse2[h, lo:hi] - ref2).max() <= 2.0 ** -8 / np.log(2.0) + 1e-4
    # the two-phase call continues a state in one of the slices
    b = lf.lf_chunk_budget(w.chunk_idx, w.schedule)
    idx = lf.lf_select_mask(Q, K, w.frame_len, w.block, b)
    one = lf.lf_sparse_attn(Q, K, V, idx, w.frame_len, w.block)
    two = lf.lf_sparse_attn_split(Q, K, V, idx, w.frame_len, w.block, b)
    torch.cuda.synchronize()
    diff = (one.float() - two.float()).abs()
    assert float(diff.max()) <= 2 * MAX_ABS and float(diff.mean()) <= 2 * MEAN_ABS


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("heads,frame_len,chunk", [(2, 256, 4), (2, 257, 4), (1, 512, 5), (3, 193, 4), (2, 64, 6), (2, 1, 6),
                                                   (16, 65, 16), (16, 65, 17), (8, 64, 16), (8, 64, 17)])
def test_short_frames_pooled_in_one_launch(gpu, heads, frame_len, chunk, head_dim):
    """Block and frame means of short frames come from one launch: frames of 1, 2 and 4 blocks (full
    and short last ones) and of 5 and 8, which take two launches; 512 and 544 frames in all (of one
    block: 256 and 272); the same through the pooled-key cache."""
    torch, lf = gpu
    w = synth.small_ragged(frame_len=frame_len, chunk_idx=chunk, heads=heads, head_dim=head_dim, n_win=1)
    x = synth.make_inputs(w)
    print(f"short frames: heads={heads} d={head_dim} n={frame_len} frames={w.frames}", flush=True)
    dev, idx, lists = _run_select(torch, lf, w, x)[:3]
    Q, K = dev[0], dev[1]
    b = lf.lf_chunk_budget(w.chunk_idx, w.schedule)
    sh = lf.make_shape(Q, K, frame_len=w.frame_len, block=w.block)
    cache = torch.zeros(lf.lf_kcache_bytes(sh, w.frames), dtype=torch.uint8, device="cuda")
    lf.lf_kcache_update(K, w.frame_len, w.block, 0, w.frames, w.frames, cache)
    again = lf.lf_select_mask_cached(Q, cache, w.frames, w.kv_len, w.frame_len, w.block, b)
    torch.cuda.synchronize()
    assert np.array_equal(again.cpu().numpy(), idx.cpu().numpy())


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("frame_len,keep", [(200, 40), (129, 11)])
def test_a_head_gives_the_same_whether_its_lists_are_divided_or_not(gpu, frame_len, keep, head_dim):
    """The first heads of a call with many query blocks (undivided lists) against a call with these
    heads alone (divided), forward in one and in two phases, and the training pair.  Both forms
    round the probabilities against the same reference, so O differs only by the order of float32 sums:
    at most S = 4 * keep products are added into an element, each sum off by at most 2^-24 of the largest
    partial one, which the typical case passes by far less (sqrt(S) 2^-24 = 8e-7 of |O|).  Against the spacing of
    bfloat16 values (2^-8 |O| or more) that moves fewer than one in a hundred elements, by one
    spacing (2^-7 |O| at most).  With a reference per slice about one in three moves."""
    torch, lf = gpu
    heads, few = 600 // (2 * -(-frame_len // 64)) + 1, 3
    w = synth.small_ragged(frame_len=frame_len, chunk_idx=6, heads=heads, head_dim=head_dim)
    x = synth.make_inputs(w)
    x["dO"] = synth.make_upstream_grad(w)
    Q, K, V, dO = (_dev(torch, x[k]) for k in ("Q", "K", "V", "dO"))
    n_q, n_k, cur = (v * w.blocks_per_frame for v in (w.frames_per_chunk, w.frames, w.frames_per_chunk))
    rng = np.random.default_rng(keep)
    pick = min(keep, n_k - cur)
    lists = np.stack([np.stack([np.concatenate([np.sort(rng.choice(n_k - cur, pick, replace=False)),
                                                np.arange(n_k - cur, n_k)]) for _ in range(n_q)])
                      for _ in range(heads)]).astype(np.int32)
    lists[0, 0, :3] = [-3, -2, -1]               # the first valid id is not the first entry
    print(f"divided or not: heads={heads} d={head_dim} n={frame_len} L={lists.shape[-1]}", flush=True)
    idx = torch.from_numpy(lists).cuda()
    b = lf.lf_chunk_budget(w.chunk_idx, w.schedule)
    b.n_sink = b.n_win = 0
    b.k_frames, b.k_blocks, b.list_len = w.hist_frames, pick, lists.shape[-1]

    def calls(hs):
        q, k, v, g, i = (t[:hs].contiguous() for t in (Q, K, V, dO, idx))
        out, lse2 = lf.lf_sparse_attn_fwd(q, k, v, i, w.frame_len, w.block)
        two = lf.lf_sparse_attn_split(q, k, v, i, w.frame_len, w.block, b)
        grads = lf.lf_sparse_attn_bwd(q, k, v, out, g, lse2, i, w.frame_len, w.block)
        torch.cuda.synchronize()
        return (out, two) + grads, lse2
    (many, lse_many), (alone, lse_alone) = calls(heads), calls(few)
    for name, a, c in zip(("O", "O in two phases", "dQ", "dK", "dV"), many, alone):
        a, c = a[:few].double(), c.double()
        share = float((a != c).double().mean())
        print(f"  {name}: {share:.2e} of the elements differ", flush=True)
        if name.startswith("O"):
            assert share <= 1e-2 and bool(((a - c).abs() <= 2.0 ** -7 * c.abs() + 1e-6).all()), (name, share)
        else:
            # O's rare steps reach the gradients through delta = dO . O: less than a spacing on average
            assert float((a - c).norm() / c.norm()) <= 5e-4, name
    # log2 of a float32 sum of keep * 64 probabilities, in another order
    assert float((lse_many[:few] - lse_alone).abs().max()) <= 1.5 * keep * 64 * 2.0 ** -24 + 2.0 ** -20


def test_the_place_of_the_v_request_does_not_change_a_bit(gpu):
    """Whole frames at d = 128: 512, 520 and 1 024 query blocks and 1 032, where the kernel asks for V
    late, early, early and late.  The heads that all calls share give the same bits, and sampled
    blocks of them match the oracle."""
    torch, lf = gpu
    w = synth.small_ragged(frame_len=256, chunk_idx=3, heads=129, head_dim=128)
    x = synth.make_inputs(w)
    Q, K, V = (_dev(torch, x[k]) for k in "QKV")
    n_q, n_k, L = w.frames_per_chunk * w.blocks_per_frame, w.frames * w.blocks_per_frame, 13
    rng = np.random.default_rng(1)
    lists = rng.integers(-1, n_k + 1, (w.heads, n_q, L)).astype(np.int32)
    outs = []
    for heads in (64, 65, 128, 129):
        print(f"place of the V request: {heads * n_q} query blocks", flush=True)
        idx = torch.from_numpy(lists[:heads]).cuda()
        outs.append(lf.lf_sparse_attn(Q[:heads], K[:heads], V[:heads], idx, w.frame_len, w.block)[:64])
    torch.cuda.synchronize()
    for o in outs[1:]:
        assert torch.equal(o.view(torch.int16), outs[0].view(torch.int16))
    got = outs[0].float().cpu().numpy().astype(np.float64)
    Qf, Kf, Vf = (_host_f32(x[k][:64]) for k in "QKV")
    for h, r in ((0, 0), (63, n_q - 1), (31, 3)):
        kept = [int(c) for c in lists[h, r] if 0 <= c < n_k]
        lo, hi = O.block_token_range(r, w.frame_len, w.block)
        err = np.abs(got[h, lo:hi] - O.sparse_attention_block(Qf[h], Kf[h], Vf[h], r, kept, w.frame_len, w.block))
        assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS, (h, r, err.max())


def _mixed_lists(w, heads, L, rng):
    """[heads, n_q, L]: neighbours differ in their number of half tiles (only short tail blocks, only full
    ones, a mix with ids out of range, hardly any valid id, and per head one list without any)."""
    nb, n_q, n_k = w.blocks_per_frame, w.frames_per_chunk * w.blocks_per_frame, w.frames * w.blocks_per_frame
    ids = np.arange(n_k, dtype=np.int32)
    lists = rng.integers(-2, n_k + 2, (heads, n_q, L)).astype(np.int32)
    for h in range(heads):
        for r in range(n_q):
            kind = (r + h) % 4
            if kind == 0:
                lists[h, r] = rng.choice(ids[ids % nb == nb - 1], L)
            elif kind == 1:
                lists[h, r] = rng.choice(ids[ids % nb != nb - 1], L)
            elif kind == 3:
                lists[h, r] = -1
                lists[h, r, rng.integers(0, L)] = rng.integers(0, n_k)
        lists[h, h % n_q] = n_k
    return lists


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("heads,lengths", [(130, (255, 256, 257, 513)), (260, (255, 256, 257, 513)), (2, (511, 512, 513, 1024, 1025))])
def test_list_lengths_around_the_decode_passes(gpu, heads, lengths, head_dim):
    """Lists are decoded 256 entries per pass where every pair of wavefronts has a query block of its own (260
    heads, 1 040 query blocks; at d = 64 also 130 heads, 520), 512 where every wavefront has one (130 heads at
    d = 128) and 128 entries of each quarter where they are divided (2 heads, 8 query blocks): lengths
    around one and two passes, on lists whose numbers of half tiles differ between
    the query blocks of a workgroup, from tensors carved out of larger ones, also into guarded memory."""
    torch, lf = gpu
    w = synth.small_ragged(frame_len=72, chunk_idx=4, heads=heads, head_dim=head_dim)
    x = synth.make_inputs(w)
    Qf, Kf, Vf = (_host_f32(x[k]) for k in "QKV")

    def strided(bits, value):
        H, L, d = bits.shape
        buf = torch.full((H, L + 5, d + 8), value, dtype=torch.bfloat16, device="cuda")
        view = buf[:, 2:2 + L, :d]
        view.copy_(_dev(torch, bits))
        return buf, view
    (_, Q), (_, K), (_, V), (Obuf, Oview) = (strided(x[k], float("nan")) for k in "QKVQ")
    rng = np.random.default_rng(heads)
    n_q, n_k = w.frames_per_chunk * w.blocks_per_frame, w.frames * w.blocks_per_frame
    for L in lengths:
        print(f"decode passes: heads={heads} d={head_dim} list length {L}", flush=True)
        lists = _mixed_lists(w, heads, L, rng)
        idx = torch.from_numpy(lists).cuda()
        out = lf.lf_sparse_attn(Q, K, V, idx, w.frame_len, w.block, O=Oview)
        torch.cuda.synchronize()
        got = out.float().cpu().numpy().astype(np.float64)
        assert np.isfinite(got).all()
        again = lf.lf_sparse_attn(Q, K, V, idx, w.frame_len, w.block, O=torch.empty_like(Oview))
        assert torch.equal(again.view(torch.int16), out.view(torch.int16))
        for h in sorted({0, 1, heads // 2, heads - 1}):
            for r in range(n_q):
                kept = [int(c) for c in lists[h, r] if 0 <= c < n_k]
                lo, hi = O.block_token_range(r, w.frame_len, w.block)
                if not kept:
                    assert np.all(got[h, lo:hi] == 0.0)
                    continue
                ref = O.sparse_attention_block(Qf[h], Kf[h], Vf[h], r, kept, w.frame_len, w.block)
                err = np.abs(got[h, lo:hi] - ref)
                assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS, (L, h, r, err.max())
    # nothing outside the O view was touched
    assert torch.isnan(Obuf[:, :2].float()).all() and torch.isnan(Obuf[:, 2 + w.q_len:].float()).all()
    assert torch.isnan(Obuf[:, :, w.head_dim:].float()).all()


@pytest.mark.parametrize("scale", [0.25, 1.0, 4.0])
@pytest.mark.parametrize("frame_len,head_dim,heads,chunk", [(200, 128, 66, 4), (256, 128, 66, 4), (200, 64, 66, 4),
                                                            (200, 128, 132, 4), (256, 128, 66, 3)])
def test_extreme_logits_with_many_query_blocks(gpu, frame_len, head_dim, heads, chunk, scale):
    """test_attention_with_extreme_logits on many query blocks, where each list is walked by one pair of wavefronts
    (d = 64; 1 056 query blocks) or by one wavefront (528): the reference
    moves inside the list."""
    torch, lf = gpu
    w = synth.small_ragged(frame_len=frame_len, chunk_idx=chunk, heads=heads, head_dim=head_dim)
    x = synth.make_inputs(w)
    n = w.frame_len
    Kf = _host_f32(x["K"]).copy()
    Kf[:, 0:n] *= 0.05          # a first frame with tiny logits, then much larger ones
    Kf[:, 2 * n:3 * n] *= 3.0
    K = synth.f32_to_bf16_bits(Kf)
    lists = O.full_lists(w.heads, n, w.block, w.frames_per_chunk, w.frames)
    print(f"extreme logits, many query blocks: n={n} d={head_dim} scale {scale}", flush=True)
    out = lf.lf_sparse_attn(_dev(torch, x["Q"]), _dev(torch, K), _dev(torch, x["V"]), torch.from_numpy(lists).cuda(),
                            n, w.block, softmax_scale=scale)
    torch.cuda.synchronize()
    got = out.float().cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all()
    Qf, Kf, Vf = _host_f32(x["Q"]), _host_f32(K), _host_f32(x["V"])
    for h in (0, heads // 2, heads - 1):
        for r in range(lists.shape[1]):
            lo, hi = O.block_token_range(r, n, w.block)
            ref = O.sparse_attention_block(Qf[h], Kf[h], Vf[h], r, list(lists[h, r]), n, w.block, scale=scale)
            err = np.abs(got[h, lo:hi] - ref)
            assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS, (h, r, err.max(), err.mean())


# One wavefront per query block (d = 128, lists of 32 and more, 513 to 1 024 query blocks or 1 792: a second round of 768) at its
# edges: blocks of 1, 31, 32, 33 and 64 tokens, lists with 0, 1, 2, 3 valid ids and with odd and even numbers of half
# tiles, more entries than a pass decodes (512), the log-sum-exp beside it.
@pytest.mark.parametrize("frame_len,list_len,heads", [(31, 33, 9), (64, 32, 9), (65, 47, 9), (96, 48, 9), (97, 40, 9), (64, 515, 9),
                                                      (33, 1030, 9), (31, 33, 28), (65, 47, 28)])
def test_one_wavefront_per_query_block(gpu, frame_len, list_len, heads):
    torch, lf = gpu
    nb = -(-frame_len // 64)
    f = 64 // nb
    F = max(f, -(-list_len // nb))
    rng = np.random.default_rng(frame_len)
    mk = lambda t: synth.f32_to_bf16_bits(rng.standard_normal((heads, t * frame_len, 128), dtype=np.float32))
    x = {"Q": mk(f), "K": mk(F), "V": mk(F)}
    n_q, n_k = f * nb, F * nb
    assert heads * n_q in (576, 1792)
    lists = np.stack([[rng.permutation(n_k)[:list_len] for _ in range(n_q)] for _ in range(heads)])
    lists = np.pad(lists, ((0, 0), (0, 0), (0, list_len - lists.shape[2])), constant_values=-1)
    for r in range(4):                 # few valid ids, at the list's end and beginning
        lists[0, r, : list_len - r] = -1
        lists[1, r, r:] = n_k
    lists[2, 0, ::2] = -1
    x["Q"][8, 5] = 0x7FC0              # a NaN row stays in its row
    Q, K, V = (_dev(torch, x[k]) for k in "QKV")
    idx = torch.from_numpy(lists.astype(np.int32)).cuda()
    out, lse2 = lf.lf_sparse_attn_fwd(Q, K, V, idx, frame_len, 64)
    got = out.float().cpu().numpy()
    assert torch.equal(out.view(torch.int16), lf.lf_sparse_attn(Q, K, V, idx, frame_len, 64).view(torch.int16))
    assert np.isnan(got[8, 5]).all()
    got[8, 5] = 0.0
    assert np.isfinite(got).all()
    Qf, Kf, Vf = (_host_f32(x[k]) for k in "QKV")
    for h, r in [(0, 0), (0, 1), (0, 2), (0, 3), (1, 0), (1, 1), (1, 2), (1, 3), (2, 0), (8, 0), (8, n_q - 1), (5, n_q // 2), (heads - 1, 1)]:
        kept = [c for c in lists[h, r] if 0 <= c < n_k]
        lo, hi = O.block_token_range(r, frame_len, 64)
        if not kept:
            assert not got[h, lo:hi].any() and np.isinf(lse2[h, lo:hi].cpu().numpy()).all()
            continue
        ref = O.sparse_attention_block(Qf[h], Kf[h], Vf[h], r, kept, frame_len, 64)
        if h == 8 and lo <= 5 < hi:
            ref[5 - lo] = 0.0
        err = np.abs(got[h, lo:hi] - ref)
        assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS, (h, r, err.max(), err.mean())
    again = [lf.lf_sparse_attn(Q, K, V, idx, frame_len, 64).view(torch.int16) for _ in range(5)]
    assert all(torch.equal(a, again[0]) for a in again)


@pytest.mark.parametrize("frame_len", [200, 256, 161])
def test_one_wavefront_per_query_block_continues_a_state(gpu, frame_len):
    """The list-driven phase after the dense one over the current chunk, on 544 to 576 query blocks."""
    torch, lf = gpu
    nb = -(-frame_len // 64)
    w = synth.small_ragged(frame_len=frame_len, chunk_idx=8, heads=-(-544 // (2 * nb)), keep_fixed=0.9, k_frames=10)
    x = synth.make_inputs(w)
    b = lf.lf_chunk_budget(w.chunk_idx, w.schedule)
    n_q = w.frames_per_chunk * nb
    assert b.current_mandatory == 1 and b.k_blocks >= 32 and 512 < w.heads * n_q <= 1024
    Q, K, V = (_dev(torch, x[k]) for k in "QKV")
    idx = lf.lf_select_mask(Q, K, frame_len, w.block, b)
    got = lf.lf_sparse_attn_split(Q, K, V, idx, frame_len, w.block, b).float().cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all()
    lists = idx.cpu().numpy()
    for h, r in ((0, 0), (0, n_q - 1), (w.heads // 2, nb - 1), (w.heads - 1, n_q - 1)):
        lo, hi = O.block_token_range(r, frame_len, w.block)
        ref = O.sparse_attention_block(*(_host_f32(x[k][h]) for k in "QKV"), r, [int(c) for c in lists[h, r]], frame_len, w.block)
        err = np.abs(got[h, lo:hi] - ref)
        assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS, (h, r, err.max(), err.mean())
