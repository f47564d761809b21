"""Parity of the Q/K producer kernel (RMSNorm + rotary embedding, head-major output) with its
binary64 oracle, through the C ABI.

Bar: the kernel computes in float32 and rounds once to bfloat16, so against the binary64 result
every element is within one bfloat16 unit in the last place (2^-7 relative; half a unit is the
rounding itself, the other half covers float32 results that fall next to a rounding boundary),
at most one element in a thousand differs from the correctly rounded oracle value at all, and
nothing is written outside the addressed rows."""
import numpy as np
import pytest

from oracle import qk_producer_oracle as P
from paper_2602_04789_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_04789_amd import lf
    lf.load()
    return torch, lf


def _check(torch, lf, L, H, d, seed, across, pairing, rows=None, x_pad=0, into_cache=False):
    x = synth.make_producer_inputs(L, H, d, seed, x_pad=x_pad)
    X = torch.from_numpy(x["X"]).view(torch.bfloat16).cuda()
    g, c, s = (torch.from_numpy(x[k]).cuda() for k in ("g", "cos", "sin"))
    if into_cache:     # Y is the last L tokens of a larger [H, L + 11, d + 8] buffer filled with NaN
        buf = torch.full((H, L + 11, d + 8), float("nan"), dtype=torch.bfloat16, device="cuda")
        Y = buf[:, 11:, :d]
    else:
        buf = None
        Y = torch.empty((H, L, d), dtype=torch.bfloat16, device="cuda")
    lf.lf_qk_norm_rope(X, g, c, s, H, Y, eps=1e-6, across_heads=across, pairing=pairing)
    torch.cuda.synchronize()
    got = Y.float().cpu().numpy().astype(np.float64)
    rows = np.arange(L) if rows is None else np.asarray(rows)
    xf = synth.bf16_bits_to_f32(x["X"])[rows, :H * d]
    ref = P.qk_norm_rope(xf, x["g"], x["cos"][rows], x["sin"][rows], H, eps=1e-6,
                         across_heads=bool(across), pairing="interleaved" if pairing == 0 else "half")
    err = np.abs(got[:, rows] - ref)
    assert np.all(err <= 2.0 ** -7 * np.abs(ref) + 1e-30), float((err / (np.abs(ref) + 1e-30)).max())
    rounded = synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(ref.astype(np.float32))).astype(np.float64)
    assert np.mean(got[:, rows] != rounded) <= 1e-3
    if buf is not None:
        assert torch.isnan(buf[:, :11].float()).all() and torch.isnan(buf[:, :, d:].float()).all()
    return float((err / (np.abs(ref) + 1e-30)).max())


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("across", [0, 1])
@pytest.mark.parametrize("pairing", [0, 1])
def test_small_cases_every_element(gpu, d, across, pairing):
    torch, lf = gpu
    # 37 tokens (a ragged last workgroup), 3 and 5 heads (chunks per token not a multiple of 64)
    for H, L, pad, cache in ((3, 37, 0, False), (5, 130, 24, True)):
        print(f"producer case d={d} across={across} pairing={pairing} H={H} L={L}", flush=True)
        _check(torch, lf, L, H, d, seed=d + across + pairing, across=across, pairing=pairing,
               x_pad=pad, into_cache=cache)


@pytest.mark.parametrize("heads", [12, 40])
def test_chunk_sized_call_on_sampled_tokens(gpu, heads):
    """One chunk of the benchmark shape (3 frames of 1560 tokens, 128 channels per head), the
    oracle evaluated on 96 sampled tokens (rows are independent of each other)."""
    torch, lf = gpu
    L = 4680
    rows = np.unique(np.concatenate([[0, 1, 1559, 1560, L - 1],
                                     np.random.default_rng(heads).integers(0, L, 91)]))
    worst = _check(torch, lf, L, heads, 128, seed=heads, across=0, pairing=0, rows=rows, into_cache=True)
    _check(torch, lf, L, heads, 128, seed=heads + 1, across=1, pairing=1, rows=rows)
    print(f"producer {heads} heads: worst relative error {worst:.2e}", flush=True)


@pytest.mark.parametrize("across", [0, 1])
@pytest.mark.parametrize("heads,d", [(16, 128), (17, 128), (48, 128), (49, 128), (96, 64), (97, 64)])
def test_token_lengths_around_the_register_forms(gpu, heads, d, across):
    """Tokens of 256, 272, 768 and 784 chunks (of 8 channels): the last and first ones of the forms
    that hold 4 x 64 and 12 x 64 chunks in registers and of the one that reads a token twice."""
    torch, lf = gpu
    print(f"producer case heads={heads} d={d} across={across}", flush=True)
    _check(torch, lf, 9, heads, d, seed=heads, across=across, pairing=across, x_pad=8, into_cache=True)


def test_binding_rejects_bad_arguments(gpu):
    torch, lf = gpu
    x = synth.make_producer_inputs(8, 2, 64, 0)
    X = torch.from_numpy(x["X"]).view(torch.bfloat16).cuda()
    g, c, s = (torch.from_numpy(x[k]).cuda() for k in ("g", "cos", "sin"))
    Y = torch.empty((2, 8, 64), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(ValueError):
        lf.lf_qk_norm_rope(X, g, c[:, :16].contiguous(), s, 2, Y)
    with pytest.raises(lf.LfError):
        lf.lf_qk_norm_rope(X, g, c, s, 2, Y, eps=-1.0)
