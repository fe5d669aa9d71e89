"""Kept sets, kept rows and the ring where a head's selection is shared out over several workgroups: two to eight slices of 64 rows and
more, heads that keep fewer entries than there are slices' rows, segments one longer and one shorter than a multiple, continued
prefills (which read the old count while another slice sets the new one).  Bars as in test_gpu_append."""
import numpy as np
import pytest

from tests import test_gpu_append as base

pytestmark = pytest.mark.gpu

CNN = ((5,), (32,), None)
CASES = {
    "slices_eight": ([1400], 1, 1, 64, 64, 512, 0, -np.inf, *CNN, [0.6]),
    "slices_eight_and_one": ([1301, 90], 2, 1, 64, 40, 513, 2, 0.0, *CNN, [0.5, 0.9]),
    "slices_two": ([700, 333], 4, 2, 64, 64, 127, 0, -np.inf, *CNN, [0.4]),
    "slices_partly_filled": ([900], 2, 2, 128, 300, 640, 1, 0.05, *CNN, [0.7]),
}


@pytest.mark.parametrize("name", list(CASES))
def test_slices(name, monkeypatch):
    monkeypatch.setitem(base.CASES, name, CASES[name])
    base.test_append_equals_one_shot_prefill(name)
