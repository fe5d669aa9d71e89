"""The decode step's scoring role for stacks against the oracle where its rows and column tiles can go wrong: every number of 16-channel
tiles per layer, two and three layers, one sequence and one more than two groups, windows no longer than the receptive field allows,
tokens whose receptive field begins before the sequence.  Bars as in test_gpu_decode_roles."""
import pytest

from tests import test_gpu_decode_roles as base

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("channels,dilation,lens", [
    ((64, 64, 64), 1, [90]),
    ((32, 64, 32), 2, [1, 7, 90]),
    ((64, 32, 16), 7, [43, 44, 100]),                # window 48 and a reach of 21 to either side
    ((32, 16), 3, [80, 3]),
    ((64, 64), 1, [i * 5 for i in range(17)]),
    ((64, 16), 11, [70, 46]),
])
def test_stack_role(channels, dilation, lens):
    n = len(channels)
    base.test_eager_step("bf16", 4, 2, 64, ((3,) * n, channels, (dilation,) * n), lens)
