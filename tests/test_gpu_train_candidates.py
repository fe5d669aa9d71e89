"""Training forward / backward against the oracle where few of a row's keys are in its window and most are candidates: more
than 64 of them (the search for the last one that a block of queries sees takes several steps), windows that end inside a
block of 32 keys or at one, query rows before the first candidate, sequences of one tile and with one token past it.  Bars as in
test_gpu_train."""
import pytest

from tests import test_gpu_train as base

pytestmark = pytest.mark.gpu

CNN = ((5,), (32,), None, 0.2)
SHAPES = {
    # name: (seqlens, Hq, Hkv, D, window, sink)
    "by_head_d64": ([700, 65, 34], 4, 1, 64, 33, 2),
    "by_head_d64_aligned": ([513, 64], 8, 2, 64, 64, 0),
    "by_head_d128": ([450, 97], 4, 1, 128, 31, 1),
    "even_d64": ([611, 32], 2, 2, 64, 96, 0),
    "even_d128": ([385, 130], 2, 2, 128, 65, 3),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_train_backward_candidates(name, monkeypatch):
    monkeypatch.setitem(base.CASES, name, ("bf16", *SHAPES[name], *CNN))
    base.test_train_forward_backward(name)
