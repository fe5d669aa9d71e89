"""Training forward / backward against the oracle where the backward's tiles can go wrong: windows several tiles wide, so that
whole tiles lie inside every row's window (the body without masks), one query head per wave and one head per workgroup, the
last query or key of a tile, sequences one longer and one shorter than a tile.  Bars as in test_gpu_train."""
import pytest

from tests import test_gpu_train as base

pytestmark = pytest.mark.gpu

CNN = ((5,), (32,), None, 0.2)
SHAPES = {
    # name: (seqlens, Hq, Hkv, D, window, sink)
    "by_head_d64": ([511, 128, 33], 4, 1, 64, 200, 2),
    "by_head_d64_one_short": ([385, 127], 8, 2, 64, 129, 0),
    "by_head_d128": ([450, 65], 4, 1, 128, 192, 1),
    "pairs_d64": ([512, 257], 2, 1, 64, 321, 0),
    "even_d64": ([449, 64], 2, 2, 64, 192, 3),
    "even_d128": ([420, 191], 2, 2, 128, 255, 0),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_train_backward_tiles(name, monkeypatch):
    monkeypatch.setitem(base.CASES, name, ("bf16", *SHAPES[name], *CNN))
    base.test_train_forward_backward(name)
