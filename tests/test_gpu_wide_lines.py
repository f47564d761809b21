"""Calls at d = 128 on the lines where the kernels with one wavefront per query block or per role of a KV block begin."""
import numpy as np
import pytest

from oracle import hsa_oracle as O
from paper_2602_04789_amd import synth
from test_gpu_attn_bwd import _close
from test_gpu_parity import MAX_ABS, MEAN_ABS, _dev, _host_f32, gpu  # noqa: F401

pytestmark = pytest.mark.gpu


# Full rounds of 1 024 query blocks apart from 1, 248 and 448 more, and from 8 in two rounds; 513 query and KV blocks, mean list 16; 1 537 query blocks, and 1 536; 390 KV blocks with a mean list of 18; 192, of 18 (two pairs each);
# 520 KV blocks with a mean list of 15
@pytest.mark.parametrize("heads,per_chunk,frames,nb,tail,length", [(41, 1, 1, 25, 24, 16), (53, 1, 2, 24, 1, 16), (46, 2, 2, 16, 33, 32),
                                                                   (127, 1, 3, 16, 64, 17), (129, 2, 2, 8, 2, 16), (19, 3, 3, 9, 1, 16), (53, 1, 2, 29, 64, 16), (48, 1, 2, 32, 33, 16),
                                                                   (10, 2, 3, 13, 33, 27), (4, 2, 3, 16, 32, 27), (26, 1, 1, 20, 31, 15)])
def test_first_calls_of_the_wide_kernels(gpu, heads, per_chunk, frames, nb, tail, length):  # noqa: F811
    """O and the gradients of heads of the call against the oracle; the same bits in a second call."""
    torch, lf = gpu
    n = 64 * (nb - 1) + tail
    rng = np.random.default_rng(heads)
    bits = [synth.f32_to_bf16_bits(rng.standard_normal((heads, f * n, 128), dtype=np.float32)) for f in (per_chunk, frames, frames, per_chunk)]
    Q, K, V, dO = (_dev(torch, b) for b in bits)
    n_q, n_k = per_chunk * nb, frames * nb
    lists = np.stack([np.sort(rng.permutation(n_k)[:length]) for _ in range(heads * n_q)]).astype(np.int32).reshape(heads, n_q, length)
    print(f"first calls: {heads * n_q} query blocks, {heads * n_k} KV blocks, lists of {length}", flush=True)
    idx = torch.from_numpy(lists).cuda()

    def call():
        out, lse2 = lf.lf_sparse_attn_fwd(Q, K, V, idx, n, 64)
        return (out,) + tuple(lf.lf_sparse_attn_bwd(Q, K, V, out, dO, lse2, idx, n, 64))
    runs = [call(), call()]
    for a, b in zip(*runs):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    got = [t.float().cpu().numpy().astype(np.float64) for t in runs[0]]
    for h in sorted({0, min(1024 // n_q, heads - 1), heads - 1}):
        q, k, v, g = (_host_f32(b[h:h + 1]) for b in bits)
        err = np.abs(got[0][h:h + 1] - O.sparse_attention(q, k, v, lists[h:h + 1], n, 64))
        assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS, (h, err.max(), err.mean())
        for name, t, ref in zip(("dQ", "dK", "dV"), got[1:], O.sparse_attention_backward(q, k, v, g, lists[h:h + 1], n, 64)):
            _close(name, t[h:h + 1], ref)
