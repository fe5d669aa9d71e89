"""Scoring by the LDS-operand kernel against the oracle where its tiles can go wrong: one token more or less than a tile of 128
or 256 tokens and than a group of 2, 4, 5 and 8 of them, both forms of the kernel, both head sizes, every kernel size and the widest
reach, fewer channels than a matrix tile, sequences without a whole tile, many short ones.  Bars as in test_gpu_parity."""
import pytest

from oracle import ltea_oracle as orc
from paper_2510_20787_amd import binding as B
from paper_2510_20787_amd import workloads as wl
from tests.gpu_util import DeviceWorkload, to_np
from tests.helpers import oracle_cnn
from tests.test_gpu_parity import logit_eps

pytestmark = pytest.mark.gpu

SHORT = [(i * 37) % 130 for i in range(70)]
EDGES = [4096 + 1, 4096, 4096 - 1, 5]                # of groups of 2, 4 and 8 tiles of either size
# ..., waves of 32 tokens per tile, tiles per workgroup, single-tile form: what the rule picks (test_score_groups holds it to this)
CASES = [
    (128, 3, 1, 32, 1, [129, 1, 0, 300], (4, 1, True)),
    (128, 8, 3, 24, 4, [1025, 127, 128], (4, 1, True)),
    (128, 2, 5, 32, 1, [1024 + 1, 1024, 1023, 5, 128 + 1], (4, 1, True)),
    (128, 9, 5, 32, 2, [2300, 70], (4, 1, True)),
    (128, 2, 7, 32, 1, [2048 + 1, 2048, 2047, 3, 256 + 1, 255], (4, 1, True)),
    (128, 1, 9, 7, 1, [513, 9, 64], (4, 1, True)),
    (64, 2, 7, 32, 1, [2049, 511, 2, 256], (4, 1, True)),
    (64, 8, 9, 30, 1, [700, 257], (4, 1, True)),
    (64, 3, 1, 32, 3, [1100, 128, 33], (4, 1, True)),
    (64, 8, 7, 32, 1, SHORT, (4, 1, True)),
    (64, 2, 9, 32, 1, SHORT, (4, 1, True)),
    (64, 2, 1, 9, 1, SHORT, (4, 1, True)),
    (128, 2, 3, 32, 3, SHORT, (4, 1, True)),
    (128, 2, 5, 32, 2, SHORT, (4, 1, True)),
    (128, 2, 7, 32, 1, SHORT, (4, 1, True)),
    (128, 8, 5, 32, 2, EDGES, (4, 2, False)),
    (128, 32, 5, 24, 1, EDGES, (4, 8, False)),
    (128, 8, 7, 32, 1, EDGES, (8, 2, False)),
    (128, 8, 9, 20, 1, EDGES, (8, 2, False)),
    (128, 16, 7, 32, 1, [12288, 2047, 2049, 1], (8, 5, False)),
    (64, 16, 7, 32, 1, EDGES, (8, 4, False)),
    (64, 16, 9, 32, 1, EDGES, (8, 4, False)),
    (64, 32, 7, 32, 1, [8 * 2048 - 1], (8, 8, False)),
    (64, 32, 9, 17, 1, [8 * 2048 - 1], (8, 8, False)),
]


@pytest.mark.parametrize("D,Hkv,kernel,channels,dilation,lens,tiling", CASES)
def test_score_tiles(D, Hkv, kernel, channels, dilation, lens, tiling):
    w = wl.make_prefill("score_tiles", 500 + D + kernel + Hkv, "bf16", lens, Hkv, Hkv, D, 64, 16, 0, 0.0, cnn_kernel=(kernel,),
                        cnn_channels=(channels,), cnn_dilation=(dilation,), qkv_scale=0.5, w_std=0.05)
    z64 = orc.score(w.k, w.v, oracle_cnn(w.cnn), w.cu_seqlens)
    d = DeviceWorkload(w)
    logit_eps(to_np(B.ltea_score(d.cfg, d.cnn, d.k, d.v, d.cu, d.max_seqlen)), z64, w.dtype)
