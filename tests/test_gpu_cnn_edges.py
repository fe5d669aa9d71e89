"""Backward of the scoring CNN against the oracle at the edges of its tiles: totals of 1, 127, 128 and 129 tokens and one past
two tiles (rows outside the buffer descriptors), channel counts that end inside a column block, a 32-channel tile, a stage
(8 and 40 of 16) or just past a block (72), one tap, and taps that reach past both ends of every sequence.  Both storage types:
the fp32 kernels share the epilogues.  Bars as in test_gpu_train."""
import pytest

from tests import test_gpu_train as base

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("kernel,channels,dilation,lens", [
    ((3,), (8,), (1,), [1]),
    ((1,), (40,), (1,), [127]),
    ((3, 1), (40, 8), (1, 1), [128]),
    ((5, 3), (72, 40), (3, 2), [1, 2, 125, 1]),
    ((3, 3, 3), (24, 72, 8), (1, 2, 4), [250, 7]),
])
def test_cnn_backward_at_tile_edges(dtype, kernel, channels, dilation, lens):
    base.test_cnn_backward(dtype, kernel, channels, dilation, lens)
