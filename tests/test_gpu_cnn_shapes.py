"""Backward of the scoring CNN against the oracle where the tap groups and the shared rows of the weight products can go wrong:
one and several groups of taps (kernel, dilation), dilations at and beyond the rows staged past a slice, every combination of
narrow and wide channel counts above the first layer, sequences shorter than a slice.  Bars as in test_gpu_train."""
import pytest

from tests import test_gpu_train as base

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel,channels,dilation,lens", [
    ((9,), (32,), (1,), [129, 64, 63]),                        # 3 + 3 + 3 taps
    ((5,), (64,), (17,), [300, 70]),                           # 17 * 4 rows would not fit, 17 * 3 do
    ((3,), (32,), (65,), [400, 131]),                          # one tap per group
    ((3, 3, 3), (64, 64, 32), (1, 8, 9), [513, 30, 100]),      # wide on both sides; rows past a slice: 16 and one too many
    ((3, 3), (32, 64), (2, 17), [200, 128]),                   # narrow to wide, one tap per group
    ((5, 5, 3), (48, 24, 20), (1, 2, 1), [90, 1, 0, 17, 33, 250]),
])
def test_cnn_backward_shapes(kernel, channels, dilation, lens):
    base.test_cnn_backward("bf16", kernel, channels, dilation, lens)
