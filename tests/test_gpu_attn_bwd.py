"""Parity of the backward pass of the blockwise sparse attention with the CPU oracle.

Bars (derived from the arithmetic: bfloat16 inputs, probabilities and score gradients rounded
to bfloat16 before the accumulating products, float32 accumulation, bfloat16 outputs): for each
of dQ, dK, dV, max |got - ref| <= 2e-2 * max(1, max |ref|) and mean |got - ref| <= 2e-3 *
max(1, rms(ref))."""
import numpy as np
import pytest

from oracle import hsa_oracle as O
from paper_2602_04789_amd import synth

pytestmark = pytest.mark.gpu

MAX_REL, MEAN_REL = 2e-2, 2e-3


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


def _f32(bits):
    return synth.bf16_bits_to_f32(bits)


def _close(name, got, ref):
    err = np.abs(got - ref)
    bar_max = MAX_REL * max(1.0, float(np.abs(ref).max()))
    bar_mean = MEAN_REL * max(1.0, float(np.sqrt((ref ** 2).mean())))
    print(f"  {name}: max err {err.max():.3e} (bar {bar_max:.3e}), mean err {err.mean():.3e} "
          f"(bar {bar_mean:.3e}), max |ref| {np.abs(ref).max():.3f}", flush=True)
    assert np.isfinite(got).all()
    assert err.max() <= bar_max and err.mean() <= bar_mean, (name, err.max(), err.mean())


def _run(torch, lf, w, x, lists, scale=0.0):
    Q, K, V = (_dev(torch, x[k]) for k in "QKV")
    dO = _dev(torch, x["dO"])
    idx = torch.from_numpy(np.ascontiguousarray(lists, dtype=np.int32)).cuda()
    out, lse2 = lf.lf_sparse_attn_fwd(Q, K, V, idx, w.frame_len, w.block, softmax_scale=scale)
    ref_out = lf.lf_sparse_attn(Q, K, V, idx, w.frame_len, w.block, softmax_scale=scale)
    dQ, dK, dV = lf.lf_sparse_attn_bwd(Q, K, V, out, dO, lse2, idx, w.frame_len, w.block,
                                       softmax_scale=scale)
    torch.cuda.synchronize()
    assert torch.equal(out, ref_out)      # the training forward is the inference forward
    return [t.float().cpu().numpy().astype(np.float64) for t in (dQ, dK, dV)], lse2.cpu().numpy()


def _oracle_lists(w, x):
    ob = O.chunk_budget(w.chunk_idx, w.schedule)
    return O.select_mask(_f32(x["Q"]), _f32(x["K"]), w.frame_len, w.block, ob)


SMALL = {
    "tiny": lambda: synth.cfg_tiny(),
    "ragged_c2": lambda: synth.small_ragged(chunk_idx=2),
    "ragged_c4": lambda: synth.small_ragged(chunk_idx=4),
    "ragged_c6_d64": lambda: synth.small_ragged(chunk_idx=6, head_dim=64, heads=2),
    "ragged_compete": lambda: synth.small_ragged(chunk_idx=4, current_mandatory=0,
                                                 ratio_of=synth.OF_ALL, keep_fixed=0.3),
    "one_token_tail": lambda: synth.small_ragged(frame_len=129, chunk_idx=3, heads=2),
    "short_frame": lambda: synth.small_ragged(frame_len=40, chunk_idx=5, heads=2, k_frames=1),
    "tail_31": lambda: synth.small_ragged(frame_len=95, chunk_idx=3, heads=2),
    "tail_33_d64": lambda: synth.small_ragged(frame_len=97, chunk_idx=3, heads=2, head_dim=64),
    # 260 one-block frames per chunk: transposed lists of 260 entries, past the 256 that the dK / dV launch
    # decodes per pass (the lists of 266 are divided here; test_dq_over_more_than_one_decode_pass has dQ's passes)
    "many_query_blocks": lambda: synth.small_ragged(frame_len=64, chunk_idx=2, frames_per_chunk=260, heads=1,
                                                    head_dim=64, k_frames=3, n_sink=1, n_win=2),
}


@pytest.mark.parametrize("name", list(SMALL))
def test_small_cases_match_oracle_everywhere(gpu, name):
    torch, lf = gpu
    w = SMALL[name]()
    x = synth.make_inputs(w)
    x["dO"] = synth.make_upstream_grad(w)
    print(f"case {name}: H={w.heads} d={w.head_dim} n={w.frame_len} F={w.frames}", flush=True)
    lists = _oracle_lists(w, x)
    (dQ, dK, dV), lse2 = _run(torch, lf, w, x, lists)
    rQ, rK, rV = O.sparse_attention_backward(_f32(x["Q"]), _f32(x["K"]), _f32(x["V"]), _f32(x["dO"]),
                                             lists, w.frame_len, w.block)
    _close("dQ", dQ, rQ)
    _close("dK", dK, rK)
    _close("dV", dV, rV)
    # the log-sum-exp the forward left: log2 of the sum of exp(s) over the row's kept columns.
    # The kernel's row sum adds the probabilities as rounded to bfloat16 (the values its second
    # product uses), each within 2^-9 of the exact one, so log2 of the sum is within
    # log2(1 + 2^-9) = 2.8e-3; float32 accumulation adds little to that.
    Qf, Kf = _f32(x["Q"]).astype(np.float64), _f32(x["K"]).astype(np.float64)
    scale = 1.0 / np.sqrt(w.head_dim)
    nq = lists.shape[1]
    for h, r in {(0, 0), (w.heads - 1, nq - 1), (w.heads // 2, nq // 2)}:
        lo, hi = O.block_token_range(r, w.frame_len, w.block)
        cols = np.concatenate([np.arange(*O.block_token_range(c, w.frame_len, w.block)) for c in lists[h, r]])
        sc = (Qf[h, lo:hi] @ Kf[h][cols].T) * scale
        m = sc.max(axis=1)
        want = (m + np.log(np.exp(sc - m[:, None]).sum(axis=1))) / np.log(2.0)
        err = np.abs(lse2[h, lo:hi] - want).max()
        assert err <= 3.5e-3, (h, r, err)


def test_full_lists_match_library_autodiff_of_dense_attention(gpu):
    """With every block listed the gradients are those of dense attention: compared with the
    framework's autodiff of its own dense attention in float32 on the GPU (an independent
    implementation of the same derivative)."""
    torch, lf = gpu
    w = synth.small_ragged(chunk_idx=3, heads=2)
    x = synth.make_inputs(w)
    x["dO"] = synth.make_upstream_grad(w)
    lists = O.full_lists(w.heads, w.frame_len, w.block, w.frames_per_chunk, w.frames)
    (dQ, dK, dV), _ = _run(torch, lf, w, x, lists)
    Q, K, V = (_dev(torch, x[k]).float().requires_grad_(True) for k in "QKV")
    out = torch.nn.functional.scaled_dot_product_attention(Q, K, V)
    out.backward(_dev(torch, x["dO"]).float())
    for name, got, ref in (("dQ", dQ, Q.grad), ("dK", dK, K.grad), ("dV", dV, V.grad)):
        _close(name, got, ref.cpu().numpy().astype(np.float64))


# The d = 128 kernel for long lists (mean transposed list of 32 and more) at its edges: odd and even numbers of half tiles,
# blocks of 1, 31, 32, 33 and 64 tokens, more query blocks per list than a pass decodes (256), blocks with two pairs of
# wavefronts (256 KV blocks and fewer) and with one (769 to 1 024 here).
LONG_LISTS = {
    "odd_two_pairs": lambda: synth.small_ragged(frame_len=33, chunk_idx=2, frames_per_chunk=91, heads=1, head_dim=128,
                                                k_frames=3, n_sink=1, n_win=2),
    "short_blocks": lambda: synth.small_ragged(frame_len=31, chunk_idx=2, frames_per_chunk=90, heads=5, head_dim=128,
                                               k_frames=3, n_sink=1, n_win=2),
    "one_token_tail": lambda: synth.small_ragged(frame_len=65, chunk_idx=2, frames_per_chunk=51, heads=1, head_dim=128,
                                                 k_frames=3, n_sink=1, n_win=2),
    "half_tail_one_pair": lambda: synth.small_ragged(frame_len=96, chunk_idx=2, frames_per_chunk=45, heads=5, head_dim=128,
                                                     k_frames=3, n_sink=1, n_win=2),
    "two_passes": lambda: synth.small_ragged(frame_len=64, chunk_idx=2, frames_per_chunk=390, heads=1, head_dim=128,
                                             k_frames=3, n_sink=1, n_win=2),
}


@pytest.mark.parametrize("name", list(LONG_LISTS))
def test_long_lists_at_d128_match_oracle(gpu, name):
    torch, lf = gpu
    w = LONG_LISTS[name]()
    x = synth.make_inputs(w)
    x["dO"] = synth.make_upstream_grad(w)
    lists = _oracle_lists(w, x)
    n_k = w.frames * w.blocks_per_frame
    print(f"case {name}: lists {lists.shape}, {n_k} KV blocks", flush=True)
    assert lists.shape[1] * lists.shape[2] >= 32 * n_k
    assert w.heads * n_k <= 256 or 768 < w.heads * n_k <= 1024
    (dQ, dK, dV), _ = _run(torch, lf, w, x, lists)
    rQ, rK, rV = O.sparse_attention_backward(_f32(x["Q"]), _f32(x["K"]), _f32(x["V"]), _f32(x["dO"]),
                                             lists, w.frame_len, w.block)
    _close("dQ", dQ, rQ)
    _close("dK", dK, rK)
    _close("dV", dV, rV)
    # blocks whose scores are -inf for every query row: probability zero, finite gradients (also beside rows
    # past a short block's count, which are loaded as zeros)
    x["Q"][..., 0] = 0x3F80      # 1
    x["K"][:, : w.frame_len, 0] = 0xFF80      # -inf
    (dQ, dK, dV), _ = _run(torch, lf, w, x, lists)
    assert np.isfinite(dV).all() and not dV[:, : w.frame_len].any() and not dK[:, : w.frame_len].any()


# The kernel for long lists against the general one, which takes the same call with a head less (13 x 64 KV blocks are 320
# past a full round of 512, 12 x 64 only 256): the sums are in the same order, so dK and dV are the same bits.  Every KV
# block is kept by `kept` query blocks: 56 to 62 half tiles of full blocks, odd numbers of them in short frames, and (64, 0):
# lists of 40 random ids, some out of range, two blocks that no list keeps and a query block without a valid id.
@pytest.mark.parametrize("frame_len,kept", [(64, 28), (64, 29), (64, 30), (64, 31), (31, 28), (31, 29), (31, 30), (31, 31),
                                            (33, 29), (64, 0), (50, 0)])
def test_long_lists_have_the_bits_of_the_general_kernel(gpu, frame_len, kept):
    torch, lf = gpu
    heads, n_k, d = 13, 64, 128
    L = kept or 40
    rng = np.random.default_rng(100 * frame_len + kept)
    x = {k: synth.f32_to_bf16_bits(rng.standard_normal((heads, n_k * frame_len, d), dtype=np.float32)) for k in ("Q", "K", "V", "dO")}
    if kept:
        lists = np.broadcast_to(np.sort((np.arange(n_k)[:, None] + np.arange(L)) % n_k, axis=1), (heads, n_k, L)).copy()
    else:
        ids = np.setdiff1d(np.arange(n_k), (5, n_k - 1))
        lists = np.stack([[np.sort(rng.choice(ids, L, replace=False)) for _ in range(n_k)] for _ in range(heads)])
        lists[:, ::3, 0], lists[:, ::2, -1] = -2, n_k + 3
        lists[1, 2] = n_k
    assert L >= 28 and (heads * n_k - 1) % 512 >= 256 > ((heads - 1) * n_k - 1) % 512
    print(f"long lists: frames of {frame_len}, {kept} query blocks a KV block", flush=True)

    def strided(bits, pad):
        view = torch.zeros((heads, bits.shape[1] + 3, d + pad), dtype=torch.bfloat16, device="cuda")[:, 1:-2, :d]
        view.copy_(_dev(torch, bits))
        return view
    Q, K, V, dO = (strided(x[k], 0 if kept else p) for k, p in (("Q", 8), ("K", 16), ("V", 24), ("dO", 40)))
    idx = torch.from_numpy(lists.astype(np.int32)).cuda()
    out, lse2 = lf.lf_sparse_attn_fwd(Q, K, V, idx, frame_len, 64, O=torch.empty_strided(dO.shape, dO.stride(), dtype=dO.dtype, device="cuda"))

    def run(H):
        grads = tuple(torch.empty_strided(t[:H].shape, t.stride(), dtype=t.dtype, device="cuda").fill_(7.0) for t in (Q, K, V))
        lf.lf_sparse_attn_bwd(Q[:H], K[:H], V[:H], out[:H], dO[:H], lse2[:H], idx[:H], frame_len, 64, grads=grads)
        return grads
    got, want = run(heads), run(heads - 1)
    for name, g, e in zip(("dQ", "dK", "dV"), got, want):
        if name != "dQ":
            assert torch.equal(g[:-1].view(torch.int16), e.view(torch.int16)), name
    for _ in range(10):
        for g, e in zip(run(heads), got):
            assert torch.equal(g.view(torch.int16), e.view(torch.int16))
    if kept:
        h = heads - 1
        refs = O.sparse_attention_backward(*(_f32(x[k][h:]) for k in ("Q", "K", "V", "dO")), lists[h:], frame_len, 64)
        for name, g, ref in zip(("dQ", "dK", "dV"), got, refs):
            _close(name, g[h:].float().cpu().numpy().astype(np.float64), ref)
            _close(name + " rows 32 to 63", *(t.reshape(n_k, frame_len, d)[:, 32:] for t in (g[h].float().cpu().numpy(), ref[0]))) \
                if frame_len > 32 else None
    else:
        for g in got[1:]:
            assert not g[:, 5 * frame_len: 6 * frame_len].any() and not g[:, (n_k - 1) * frame_len:].any()


def test_list_edge_cases_and_strided_tensors(gpu):
    """Out-of-range ids skipped; a query block whose list holds no valid id (zero dQ rows, +inf
    log-sum-exp, no contribution to dK and dV); KV blocks that no list keeps (zero dK and dV
    rows); explicit softmax scale; tensors carved out of larger buffers."""
    torch, lf = gpu
    w = synth.small_ragged(chunk_idx=3, heads=2)
    x = synth.make_inputs(w)
    x["dO"] = synth.make_upstream_grad(w)
    nb = w.blocks_per_frame
    n_q, n_k = w.frames_per_chunk * nb, w.frames * nb
    rng = np.random.default_rng(3)
    L = 6
    lists = np.empty((w.heads, n_q, L), dtype=np.int32)
    for h in range(w.heads):
        for r in range(n_q):
            keep = np.sort(rng.choice(n_k - 2, size=L - 2, replace=False)).astype(np.int32)
            lists[h, r] = np.concatenate([[-3], keep, [n_k + 5]])       # ascending, ends invalid
    lists[1, 2] = np.array([-5, -4, -3, n_k, n_k + 1, n_k + 2])         # no valid id at all
    assert not (lists == n_k - 1).any() and not (lists == n_k - 2).any()  # two blocks nobody keeps
    scale = 0.11

    def strided(bits, pad_tok, pad_ch):
        H, Lx, d = bits.shape
        buf = torch.zeros((H, Lx + pad_tok, d + pad_ch), dtype=torch.bfloat16, device="cuda")
        view = buf[:, 1:1 + Lx, :d]
        view.copy_(_dev(torch, bits))
        return view
    Q, K, V = strided(x["Q"], 3, 8), strided(x["K"], 5, 16), strided(x["V"], 2, 24)
    dO = strided(x["dO"], 4, 8)
    Oview = torch.zeros((w.heads, w.q_len + 4, w.head_dim + 8), dtype=torch.bfloat16,
                        device="cuda")[:, 1:1 + w.q_len, :w.head_dim]
    idx = torch.from_numpy(lists).cuda()
    out, lse2 = lf.lf_sparse_attn_fwd(Q, K, V, idx, w.frame_len, w.block, softmax_scale=scale, O=Oview)
    dQ, dK, dV = lf.lf_sparse_attn_bwd(Q, K, V, out, dO, lse2, idx, w.frame_len, w.block,
                                       softmax_scale=scale)
    torch.cuda.synchronize()
    assert dQ.stride() == Q.stride() and dK.stride() == K.stride() and dV.stride() == V.stride()

    valid = [[[c for c in lists[h, r] if 0 <= c < n_k] for r in range(n_q)] for h in range(w.heads)]
    Qf, Kf, Vf, dOf = (_f32(x[k]) for k in ("Q", "K", "V", "dO"))
    rQ = np.zeros(Qf.shape)
    rK, rV = np.zeros(Kf.shape), np.zeros(Vf.shape)
    for h in range(w.heads):          # the oracle takes rectangular lists: call it per query block
        for r in range(n_q):
            if not valid[h][r]:
                continue
            lo, hi = O.block_token_range(r, w.frame_len, w.block)
            one = np.zeros((1, n_q, len(valid[h][r])), dtype=np.int32)
            one[0, r] = valid[h][r]
            mask_dO = np.zeros_like(dOf[h:h + 1])
            mask_dO[0, lo:hi] = dOf[h, lo:hi]
            # other query blocks get list [0...] with a zero upstream gradient: no contribution
            a, b, c = O.sparse_attention_backward(Qf[h:h + 1], Kf[h:h + 1], Vf[h:h + 1], mask_dO, one,
                                                  w.frame_len, w.block, scale=scale)
            rQ[h, lo:hi] = a[0, lo:hi]
            rK[h] += b[0]
            rV[h] += c[0]
    g = [t.float().cpu().numpy().astype(np.float64) for t in (dQ, dK, dV)]
    _close("dQ", g[0], rQ)
    _close("dK", g[1], rK)
    _close("dV", g[2], rV)
    lo, hi = O.block_token_range(2, w.frame_len, w.block)
    assert (g[0][1, lo:hi] == 0).all() and np.isposinf(lse2[1, lo:hi].cpu().numpy()).all()
    klo, _ = O.block_token_range(n_k - 2, w.frame_len, w.block)
    assert (g[1][:, klo:] == 0).all() and (g[2][:, klo:] == 0).all()


def test_full_size_last_chunk_one_head_against_oracle(gpu):
    """The paper's 480p last chunk at full size (12 heads on the GPU, the launch the benchmark
    times); the oracle recomputes heads 0 and 7 completely."""
    torch, lf = gpu
    w = synth.cfg_last_chunk()
    x = synth.make_inputs(w)
    x["dO"] = synth.make_upstream_grad(w)
    Q, K = _dev(torch, x["Q"]), _dev(torch, x["K"])
    b = lf.lf_chunk_budget(w.chunk_idx, w.schedule)
    idx = lf.lf_select_mask(Q, K, w.frame_len, w.block, b)
    torch.cuda.synchronize()
    lists = idx.cpu().numpy()
    print(f"full size: H={w.heads} n={w.frame_len} F={w.frames} list_len={lists.shape[-1]}", flush=True)
    (dQ, dK, dV), _ = _run(torch, lf, w, x, lists)
    # every head: what holds at any size.  The rows of P sum to one, so the token sums of dV
    # equal those of dO; the rows of dS sum to zero (delta is the P-weighted mean of dP), so the
    # token sums of dK vanish.  Sums of 32 760 bfloat16-rounded terms: absolute slack below.
    dOf = _f32(x["dO"]).astype(np.float64)
    dv_err = np.abs(dV.sum(axis=1) - dOf.sum(axis=1)).max()
    dk_err = np.abs(dK.sum(axis=1)).max()
    print(f" all heads: |sum dV - sum dO| {dv_err:.3f}, |sum dK| {dk_err:.3f}", flush=True)
    assert dv_err <= 0.5 and dk_err <= 0.5
    for h in (0, 7):
        sl = slice(h, h + 1)
        rQ, rK, rV = O.sparse_attention_backward(_f32(x["Q"][sl]), _f32(x["K"][sl]), _f32(x["V"][sl]),
                                                 _f32(x["dO"][sl]), lists[sl], w.frame_len, w.block)
        print(f" head {h}", flush=True)
        _close("dQ", dQ[sl], rQ)
        _close("dK", dK[sl], rK)
        _close("dV", dV[sl], rV)


def test_rollout_call_40_heads(gpu):
    """One call of the 40-head rollout (chunk 4, the shape of the model's full attention layer):
    the token-sum properties on every head, the oracle on the first and the last head."""
    torch, lf = gpu
    w = synth.cfg_rollout(4, 1)
    x = synth.make_inputs(w)
    x["dO"] = synth.make_upstream_grad(w)
    Q, K = _dev(torch, x["Q"]), _dev(torch, x["K"])
    b = lf.lf_chunk_budget(w.chunk_idx, w.schedule)
    lists = lf.lf_select_mask(Q, K, w.frame_len, w.block, b).cpu().numpy()
    del Q, K
    print(f"rollout call: H={w.heads} n={w.frame_len} F={w.frames} list_len={lists.shape[-1]}", flush=True)
    (dQ, dK, dV), _ = _run(torch, lf, w, x, lists)
    dOf = _f32(x["dO"]).astype(np.float64)
    dv_err = np.abs(dV.sum(axis=1) - dOf.sum(axis=1)).max()
    dk_err = np.abs(dK.sum(axis=1)).max()
    print(f" all heads: |sum dV - sum dO| {dv_err:.3f}, |sum dK| {dk_err:.3f}", flush=True)
    assert dv_err <= 0.5 and dk_err <= 0.5
    for h in (0, w.heads - 1):
        sl = slice(h, h + 1)
        rQ, rK, rV = O.sparse_attention_backward(_f32(x["Q"][sl]), _f32(x["K"][sl]), _f32(x["V"][sl]),
                                                 _f32(x["dO"][sl]), lists[sl], w.frame_len, w.block)
        print(f" head {h}", flush=True)
        _close("dQ", dQ[sl], rQ)
        _close("dK", dK[sl], rK)
        _close("dV", dV[sl], rV)


def test_backward_is_reproducible(gpu):
    """No atomics, fixed summation order: two calls give the same bits."""
    torch, lf = gpu
    w = synth.small_ragged(chunk_idx=4)
    x = synth.make_inputs(w)
    x["dO"] = synth.make_upstream_grad(w)
    lists = _oracle_lists(w, x)
    Q, K, V, dO = (_dev(torch, x[k]) for k in ("Q", "K", "V", "dO"))
    idx = torch.from_numpy(lists).cuda()
    out, lse2 = lf.lf_sparse_attn_fwd(Q, K, V, idx, w.frame_len, w.block)
    a = lf.lf_sparse_attn_bwd(Q, K, V, out, dO, lse2, idx, w.frame_len, w.block)
    b = lf.lf_sparse_attn_bwd(Q, K, V, out, dO, lse2, idx, w.frame_len, w.block)
    torch.cuda.synchronize()
    for s, t in zip(a, b):
        assert torch.equal(s, t)


def test_training_step_replays_from_a_captured_graph(gpu):
    """Selection, training forward and backward captured once into a HIP graph (the library
    allocates, clears and synchronises nothing) and replayed on new inputs written into the same
    buffers, with eager work and synchronisations between the replays; every replay must equal
    the eager result bit for bit."""
    torch, lf = gpu
    w = synth.small_ragged(chunk_idx=4)
    b = lf.lf_chunk_budget(w.chunk_idx, w.schedule)
    xs = []
    for s in (11, 12, 13):
        ws_ = synth.small_ragged(chunk_idx=4, seed=s)
        x = synth.make_inputs(ws_)
        x["dO"] = synth.make_upstream_grad(ws_, seed=s)
        xs.append(x)
    Q, K, V, dO = (_dev(torch, xs[0][k]).clone() for k in ("Q", "K", "V", "dO"))
    sh = lf.make_shape(Q, K, V, Q, frame_len=w.frame_len, block=w.block)
    ws = torch.empty(lf.lf_workspace_bytes(sh, b), dtype=torch.uint8, device="cuda")
    bws = torch.empty(lf.lf_attn_bwd_workspace_bytes(sh), dtype=torch.uint8, device="cuda")
    nq = w.frames_per_chunk * w.blocks_per_frame
    idx = torch.empty((w.heads, nq, b.list_len), dtype=torch.int32, device="cuda")
    out = torch.empty_like(Q)
    lse2 = torch.empty((w.heads, w.q_len), dtype=torch.float32, device="cuda")
    grads = (torch.empty_like(Q), torch.empty_like(K), torch.empty_like(V))

    def step():
        lf.lf_select_mask(Q, K, w.frame_len, w.block, b, indices=idx, workspace=ws)
        lf.lf_sparse_attn_fwd(Q, K, V, idx, w.frame_len, w.block, O=out, lse2=lse2)
        lf.lf_sparse_attn_bwd(Q, K, V, out, dO, lse2, idx, w.frame_len, w.block, workspace=bws, grads=grads)

    step()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step()
    for x in xs[1:] + xs[:1] + xs[1:2]:
        for t, k in ((Q, "Q"), (K, "K"), (V, "V"), (dO, "dO")):
            t.copy_(_dev(torch, x[k]))
        for t in grads:
            t.fill_(7.0)
        bws.fill_(255)
        g.replay()
        torch.cuda.synchronize()
        got = [t.clone() for t in grads]
        want_idx = lf.lf_select_mask(Q, K, w.frame_len, w.block, b)
        want_out, want_lse = lf.lf_sparse_attn_fwd(Q, K, V, want_idx, w.frame_len, w.block)
        want = lf.lf_sparse_attn_bwd(Q, K, V, want_out, dO, want_lse, want_idx, w.frame_len, w.block)
        torch.cuda.synchronize()
        for a, e in zip(got, want):
            assert torch.equal(a.view(torch.int16), e.view(torch.int16))


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("heads,list_len", [(2, 5), (2, 6), (2, 7), (2, 9), (16, 31), (16, 32), (17, 32),
                                            (16, 47), (16, 48), (17, 48), (1, 47)])
def test_lists_divided_among_the_wavefronts_of_a_workgroup(gpu, heads, list_len, head_dim):
    """dQ with and without each list divided among four pairs of wavefronts (both sides of the edges
    of that rule: list lengths 6/7, at d = 128 and more than 256 query blocks 47/48; 512 and 544 query
    blocks), one head of each against the oracle."""
    torch, lf = gpu
    w = synth.small_ragged(frame_len=1000, chunk_idx=2, heads=heads, head_dim=head_dim)
    x = synth.make_inputs(w)
    x["dO"] = synth.make_upstream_grad(w)
    n_q, n_k = w.frames_per_chunk * w.blocks_per_frame, w.frames * w.blocks_per_frame
    rng = np.random.default_rng(list_len)
    lists = np.stack([np.stack([np.sort(rng.choice(n_k, list_len, replace=False)) for _ in range(n_q)])
                      for _ in range(heads)]).astype(np.int32)
    print(f"divided lists, backward: heads={heads} d={head_dim} list length {list_len}", flush=True)
    (dQ, dK, dV), _ = _run(torch, lf, w, x, lists)
    h = heads - 1
    Qf, Kf, Vf, dOf = (_f32(x[k])[h:h + 1] for k in ("Q", "K", "V", "dO"))
    ref = O.sparse_attention_backward(Qf, Kf, Vf, dOf, lists[h:h + 1], w.frame_len, w.block)
    for name, got, want in zip(("dQ", "dK", "dV"), (dQ, dK, dV), ref):
        _close(name, got[h:h + 1], want)


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("heads,list_len", [(4, 9), (4, 1), (5, 9)])
def test_few_kv_blocks_take_two_groups_of_wavefronts(gpu, heads, list_len, head_dim):
    """dK and dV with each KV block's query blocks divided between two groups of wavefronts (256 KV
    blocks, transposed lists of 0, odd and even lengths) and, at 320 KV blocks, not."""
    torch, lf = gpu
    w = synth.small_ragged(frame_len=1000, chunk_idx=2, heads=heads, head_dim=head_dim)
    x = synth.make_inputs(w)
    x["dO"] = synth.make_upstream_grad(w)
    n_q, n_k = w.frames_per_chunk * w.blocks_per_frame, w.frames * w.blocks_per_frame
    rng = np.random.default_rng(heads + list_len)
    lists = np.stack([np.stack([np.sort(rng.choice(n_k, list_len, replace=False)) for _ in range(n_q)])
                      for _ in range(heads)]).astype(np.int32)
    print(f"two groups: heads={heads} d={head_dim} list length {list_len}", flush=True)
    got, _ = _run(torch, lf, w, x, lists)
    for h in (0, heads - 1):
        Qf, Kf, Vf, dOf = (_f32(x[k])[h:h + 1] for k in ("Q", "K", "V", "dO"))
        ref = O.sparse_attention_backward(Qf, Kf, Vf, dOf, lists[h:h + 1], w.frame_len, w.block)
        for name, g, want in zip(("dQ", "dK", "dV"), got, ref):
            _close(name, g[h:h + 1], want)


@pytest.mark.parametrize("heads,frames", [(5, 1700), (8, 1025), (1, 9), (3, 2730)])
def test_every_kv_block_is_written_over_a_long_history(gpu, heads, frames):
    """The launch order of dK and dV is made from the transposed lists' lengths, a share of the (head, KV block)
    pairs per XCD, several blocks at a time by each thread: shares of 1 063, 1 025 (one more than a pass of 128
    threads takes), 2 and 1 024 blocks.  Gradients that start as garbage are written everywhere: the
    oracle's values where a list keeps the block, zeros elsewhere."""
    torch, lf = gpu
    n, d, L = 64, 64, 9
    w = synth.small_ragged(frame_len=n, frames_per_chunk=1, chunk_idx=frames, heads=heads, head_dim=d, n_chunks=frames)
    g = torch.Generator(device="cuda")
    g.manual_seed(heads)
    Q, K, V, dO = (torch.randn((heads, t, d), generator=g, device="cuda").to(torch.bfloat16)
                   for t in (n, frames * n, frames * n, n))
    rng = np.random.default_rng(frames)
    lists = np.stack([np.sort(rng.choice(frames, L, replace=False))[None] for _ in range(heads)]).astype(np.int32)
    print(f"long history: heads={heads} frames={frames}", flush=True)
    idx = torch.from_numpy(lists).cuda()
    out, lse2 = lf.lf_sparse_attn_fwd(Q, K, V, idx, n, 64)
    grads = tuple(torch.full_like(t, 7.0) for t in (Q, K, V))
    lf.lf_sparse_attn_bwd(Q, K, V, out, dO, lse2, idx, n, 64, grads=grads)
    torch.cuda.synchronize()
    dQ, dK, dV = (t.float().cpu().numpy().astype(np.float64) for t in grads)
    Qf, dOf = (t.float().cpu().numpy() for t in (Q, dO))
    for h in range(heads):
        cols = np.concatenate([np.arange(c * n, (c + 1) * n) for c in lists[h, 0]])
        rest = np.setdiff1d(np.arange(frames * n), cols)
        assert (dK[h, rest] == 0).all() and (dV[h, rest] == 0).all()
        # the kept columns alone, as a history of their own
        rows = torch.from_numpy(cols).cuda()
        Kf, Vf = (t[h, rows].float().cpu().numpy()[None] for t in (K, V))
        rQ, rK, rV = O.sparse_attention_backward(Qf[h:h + 1], Kf, Vf, dOf[h:h + 1],
                                                 np.arange(L, dtype=np.int32)[None, None], n, 64)
        for name, got, ref in (("dQ", dQ[h:h + 1], rQ), ("dK", dK[h:h + 1, cols], rK), ("dV", dV[h:h + 1, cols], rV)):
            _close(name, got, ref)


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("heads,per_chunk,frames,list_len", [(20, 26, 300, 257), (20, 26, 300, 300), (1, 2, 1100, 1026)])
def test_dq_over_more_than_one_decode_pass(gpu, heads, per_chunk, frames, list_len, head_dim):
    """dQ decodes 256 list entries per pass: 520 query blocks with lists of 257 and 300 (undivided), and 2 with
    lists of 1 026 (divided: quarters of 257).  Strided tensors, ids out of range at both ends of the
    lists, a query block without a valid id, blocks that no list keeps, an explicit scale, two calls with the same bits.
    The key-major launch has more than 256 KV blocks, so one group of wavefronts each."""
    torch, lf = gpu
    n, scale = 40, 0.1                      # one short block per frame
    w = synth.small_ragged(frame_len=n, frames_per_chunk=per_chunk, chunk_idx=1, heads=heads, head_dim=head_dim)
    g = torch.Generator(device="cuda")
    g.manual_seed(list_len)

    def strided(tokens, pad_tok, pad_ch):
        t = torch.full((heads, tokens + pad_tok, head_dim + pad_ch), float("nan"), dtype=torch.bfloat16, device="cuda")
        view = t[:, 1:1 + tokens, :head_dim]
        view.copy_(torch.randn(view.shape, generator=g, device="cuda"))
        return view
    Q, K, V = strided(per_chunk * n, 3, 8), strided(frames * n, 5, 16), strided(frames * n, 2, 24)
    dO, Oview = strided(per_chunk * n, 4, 8), strided(per_chunk * n, 4, 8)
    rng = np.random.default_rng(list_len)
    lists = np.empty((heads, per_chunk, list_len), dtype=np.int32)
    for h in range(heads):
        for r in range(per_chunk):
            keep = np.sort(rng.choice(frames - 2, list_len - 5, replace=False))
            lists[h, r] = np.concatenate([[-9, -3], keep, [frames, frames + 1, frames + 9]])
    lists[heads - 1, 1] = np.arange(list_len) - list_len       # no valid id
    print(f"dQ passes: heads={heads} d={head_dim} blocks {heads * per_chunk} list length {list_len}", flush=True)
    idx = torch.from_numpy(lists).cuda()
    out, lse2 = lf.lf_sparse_attn_fwd(Q, K, V, idx, n, 64, softmax_scale=scale, O=Oview)
    grads = [lf.lf_sparse_attn_bwd(Q, K, V, out, dO, lse2, idx, n, 64, softmax_scale=scale) for _ in range(2)]
    torch.cuda.synchronize()
    for a, b in zip(*grads):
        assert torch.equal(a.contiguous().view(torch.int16), b.contiguous().view(torch.int16))
    dQ, dK, dV = (t.float().cpu().numpy().astype(np.float64) for t in grads[0])
    h = heads - 1
    Qf, Kf, Vf, dOf = (t[h:h + 1].float().cpu().numpy() for t in (Q, K, V, dO))
    valid = np.empty((1, per_chunk), dtype=object)
    for r in range(per_chunk):
        valid[0, r] = [int(c) for c in lists[h, r] if 0 <= c < frames]
    valid[0, 1] = [0]                        # stands for no block: without an upstream gradient it adds nothing
    dOf[0, n:2 * n] = 0
    ref = O.sparse_attention_backward(Qf, Kf, Vf, dOf, valid, n, 64, scale=scale)
    for name, got, want in zip(("dQ", "dK", "dV"), (dQ, dK, dV), ref):
        _close(name, got[h:h + 1], want)
    assert (dQ[h, n:2 * n] == 0).all() and torch.isposinf(lse2[h, n:2 * n]).all()
    assert (dK[:, (frames - 2) * n:] == 0).all() and (dV[:, (frames - 2) * n:] == 0).all()


@pytest.mark.parametrize("frame_len,head_dim", [(200, 128), (256, 128), (200, 64)])
def test_training_step_with_many_query_blocks_replays(gpu, frame_len, head_dim):
    """test_training_step_replays_from_a_captured_graph on 528 query blocks, the undivided kernels: the step
    replayed from a graph on new inputs, and run twice, gives the bits of the eager step."""
    torch, lf = gpu
    w = synth.small_ragged(frame_len=frame_len, chunk_idx=3, heads=66, head_dim=head_dim)
    b = lf.lf_chunk_budget(w.chunk_idx, w.schedule)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(frame_len)
    Q, K, V, dO = (torch.empty((w.heads, t, head_dim), dtype=torch.bfloat16, device="cuda")
                   for t in (w.q_len, w.kv_len, w.kv_len, w.q_len))

    def new_inputs():
        for t in (Q, K, V, dO):
            t.copy_(torch.randn(t.shape, generator=gen, device="cuda"))
            t[t.abs() < 2.0 ** -30] = 0
    sh = lf.make_shape(Q, K, V, Q, frame_len=w.frame_len, block=w.block)
    ws = torch.empty(lf.lf_workspace_bytes(sh, b), dtype=torch.uint8, device="cuda")
    bws = torch.empty(lf.lf_attn_bwd_workspace_bytes(sh), dtype=torch.uint8, device="cuda")
    idx = torch.empty((w.heads, w.frames_per_chunk * w.blocks_per_frame, b.list_len), dtype=torch.int32, device="cuda")
    out, lse2 = torch.empty_like(Q), torch.empty((w.heads, w.q_len), dtype=torch.float32, device="cuda")
    grads = tuple(torch.empty_like(t) for t in (Q, K, V))

    def step():
        lf.lf_select_mask(Q, K, w.frame_len, w.block, b, indices=idx, workspace=ws)
        lf.lf_sparse_attn_fwd(Q, K, V, idx, w.frame_len, w.block, O=out, lse2=lse2)
        lf.lf_sparse_attn_bwd(Q, K, V, out, dO, lse2, idx, w.frame_len, w.block, workspace=bws, grads=grads)
    new_inputs()
    step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for replay in range(3):
        print(f"graph replay {replay}: n={frame_len} d={head_dim}", flush=True)
        new_inputs()
        bws.fill_(255)
        for t in grads + (out,):
            t.fill_(7.0)
        graph.replay()
        torch.cuda.synchronize()
        got = [t.clone() for t in grads + (out,)]
        for t in grads + (out,):
            t.fill_(5.0)
        step()
        torch.cuda.synchronize()
        for a, e in zip(got, grads + (out,)):
            assert torch.equal(a.view(torch.int16), e.view(torch.int16))
