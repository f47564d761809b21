"""dQ with one wavefront per query block (d = 128, more than 512 query blocks, lists of 8 and more)."""
import numpy as np
import pytest

from oracle import hsa_oracle as O
from paper_2602_04789_amd import synth
from test_gpu_attn_bwd import _close
from test_gpu_parity import _dev, _host_f32, gpu  # noqa: F401

pytestmark = pytest.mark.gpu


# Half tiles a list around 64 (a register of entries), 128 and 256 (a pass); last blocks of 1, 31, 32, 33 and 64 rows
@pytest.mark.parametrize("frame_len,length", [(64, 8), (64, 31), (64, 32), (64, 33), (64, 47), (31, 8), (31, 9), (31, 10), (32, 47), (65, 44), (96, 43),
                                              (97, 40), (161, 45), (64, 64), (64, 127), (64, 128), (64, 129), (31, 255), (31, 256), (31, 257),
                                              (97, 300)])
def test_dq_with_one_wavefront_per_query_block(gpu, frame_len, length):  # noqa: F811
    """A call of 576 query blocks against one of 1 152 with the same first heads (too few in its last round: two wavefronts per
    block, the same order of sums) and the same O, and heads of it against the oracle.  Strided tensors, ids out of range, lists with few
    valid ids or none; the same bits in every call."""
    torch, lf = gpu
    nb = -(-frame_len // 64)
    heads, per_chunk = 24, 48 // nb
    frames = max(per_chunk, -(-length // nb) + 1)
    rng = np.random.default_rng(1000 * frame_len + length)

    def strided(tokens, pad_tok, pad_ch):
        bits = synth.f32_to_bf16_bits(rng.standard_normal((heads, tokens, 128), dtype=np.float32))
        t = torch.full((heads, tokens + pad_tok, 128 + pad_ch), float("nan"), dtype=torch.bfloat16, device="cuda")
        view = t[:, 1:1 + tokens, :128]
        view.copy_(_dev(torch, bits))
        return view, _host_f32(bits)
    (Q, Qf), (K, Kf) = strided(per_chunk * frame_len, 3, 8), strided(frames * frame_len, 2, 24)
    (V, Vf), (dO, dOf) = strided(frames * frame_len, 4, 16), strided(per_chunk * frame_len, 5, 8)
    Oview, _ = strided(per_chunk * frame_len, 5, 8)
    n_q, n_k = per_chunk * nb, frames * nb
    assert heads * n_q == 1152
    lists = np.full((heads, n_q, length), n_k + 3, dtype=np.int32)
    for h in range(heads):
        for r in range(n_q):
            lists[h, r] = np.sort(rng.permutation(n_k)[:length])
    lists[0, 0, 1:] = n_k                      # one valid id
    lists[0, 1, :-2] = -1                      # two, at the end
    lists[0, 2] = -5                           # none
    lists[0, 3, : length // 2] = -1
    print(f"dQ, one wavefront per block: n={frame_len} list length {length}", flush=True)
    idx = torch.from_numpy(lists).cuda()

    _, lse2 = lf.lf_sparse_attn_fwd(Q, K, V, idx, frame_len, 64, O=Oview)

    def call(hs):
        q, k, v, g, o, i, l = (t[:hs] for t in (Q, K, V, dO, Oview, idx, lse2))
        return [lf.lf_sparse_attn_bwd(q, k, v, o, g, l.contiguous(), i.contiguous(), frame_len, 64)[0].clone() for _ in range(3)]
    runs = call(heads // 2)
    assert all(torch.equal(m.view(torch.int16), runs[0].view(torch.int16)) for m in runs[1:])
    got = runs[0].float().cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all()
    lo, hi = O.block_token_range(2, frame_len, 64)
    assert not got[0, lo:hi].any()
    both = call(heads)[0][:heads // 2]
    assert torch.equal(runs[0].contiguous().view(torch.int16), both.contiguous().view(torch.int16))
    for h in (0, heads // 2 - 1):
        kept = np.empty((1, n_q), dtype=object)
        g = dOf[h:h + 1].copy()
        for r in range(n_q):
            kept[0, r] = [int(c) for c in lists[h, r] if 0 <= c < n_k] or [0]
            if (lists[h, r] < 0).all():
                g[0, slice(*O.block_token_range(r, frame_len, 64))] = 0     # no block: nothing is asked of it
        ref = O.sparse_attention_backward(Qf[h:h + 1], Kf[h:h + 1], Vf[h:h + 1], g, kept, frame_len, 64)
        _close("dQ", got[h:h + 1], ref[0])
