"""Scoring by the LDS-operand kernel against the oracle where its tiles can go wrong: one token more or less than a tile of 128
(k <= 5, and single tiles) or 256 tokens, both head sizes, every kernel size and the widest reach, fewer channels than a matrix tile,
sequences without a whole tile, many short ones.  Bars as in test_gpu_parity."""
import pytest

from oracle import ltea_oracle as orc
from paper_2510_20787_amd import binding as B
from paper_2510_20787_amd import workloads as wl
from tests.gpu_util import DeviceWorkload, to_np
from tests.helpers import oracle_cnn
from tests.test_gpu_parity import logit_eps

pytestmark = pytest.mark.gpu

SHORT = [(i * 37) % 130 for i in range(70)]


@pytest.mark.parametrize("D,Hkv,kernel,channels,dilation,lens", [
    (128, 3, 1, 32, 1, [129, 1, 0, 300]),
    (128, 8, 3, 24, 4, [1025, 127, 128]),
    (128, 2, 5, 32, 1, [1024 + 1, 1024, 1023, 5, 128 + 1]),
    (128, 9, 5, 32, 2, [2300, 70]),
    (128, 2, 7, 32, 1, [2048 + 1, 2048, 2047, 3, 256 + 1, 255]),
    (128, 1, 9, 7, 1, [513, 9, 64]),
    (64, 2, 7, 32, 1, [2049, 511, 2, 256]),
    (64, 8, 9, 30, 1, [700, 257]),
    (64, 3, 1, 32, 3, [1100, 128, 33]),
    (64, 8, 7, 32, 1, SHORT),
    (64, 2, 9, 32, 1, SHORT),
    (64, 2, 1, 9, 1, SHORT),
    (128, 2, 3, 32, 3, SHORT),
    (128, 2, 5, 32, 2, SHORT),
    (128, 2, 7, 32, 1, SHORT),
])
def test_score_tiles(D, Hkv, kernel, channels, dilation, lens):
    w = wl.make_prefill("score_tiles", 500 + D + kernel + Hkv, "bf16", lens, Hkv, Hkv, D, 64, 16, 0, 0.0, cnn_kernel=(kernel,),
                        cnn_channels=(channels,), cnn_dilation=(dilation,), qkv_scale=0.5, w_std=0.05)
    z64 = orc.score(w.k, w.v, oracle_cnn(w.cnn), w.cu_seqlens)
    d = DeviceWorkload(w)
    logit_eps(to_np(B.ltea_score(d.cfg, d.cnn, d.k, d.v, d.cu, d.max_seqlen)), z64, w.dtype)
