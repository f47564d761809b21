"""The binding's argument checks (no GPU: stand-ins with a tensor's attributes)."""
import pytest
import torch

from paper_2602_04789_amd import lf


class Stand:
    def __init__(self, shape=(2, 8, 64), stride=(512, 64, 1), dtype=torch.bfloat16, is_cuda=True):
        self.shape, self._stride, self.dtype, self.is_cuda = torch.Size(shape), stride, dtype, is_cuda

    def stride(self, i=None):
        return self._stride if i is None else self._stride[i]

    def dim(self):
        return len(self._stride)


def test_strides_and_shape_are_those_of_make_shape():
    Q, K, V, O = Stand(), Stand((2, 24, 64), (1600, 66, 1)), Stand((2, 24, 64), (64, 128, 1)), Stand(stride=(64, 128, 1))
    got = lf._shape_of(Q, K, *(lf._strides(t, "t") for t in (Q, K, V, O)), 8, 64)
    want = lf.make_shape(Q, K, V, O, frame_len=8, block=64)
    assert [getattr(got, n) for n, _ in lf.lf_shape._fields_] == [getattr(want, n) for n, _ in lf.lf_shape._fields_]


@pytest.mark.parametrize("bad,what", [
    (dict(is_cuda=False), "t must live in GPU memory"), (dict(dtype=torch.float16), "t must be bfloat16"),
    (dict(shape=(2, 8), stride=(8, 1)), r"t must be \[H, L, d\]"), (dict(stride=(512, 1, 8)), r"t must be \[H, L, d\]")])
def test_what_check_tensor_refuses_strides_refuses_with_the_same_words(bad, what):
    for check in (lf._check_tensor, lf._strides):
        with pytest.raises(ValueError, match=what):
            check(Stand(**bad), "t")
