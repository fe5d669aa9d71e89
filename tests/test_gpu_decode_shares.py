"""The decode step where one (sequence, KV head) is streamed by several workgroups (few heads, long caches), by groups of
more than 16 query heads, and where the finishing is a launch of its own (a CNN without look-ahead, a budget that does not
fit the counting bits of ret_count): outputs, retained sets and counters against the oracle while the ring fills up and
tokens start to leave it, and with the compact segment overflowing."""
import numpy as np
import pytest
import torch

from oracle import ltea_oracle as orc
from paper_2510_20787_amd import binding as B
from paper_2510_20787_amd import workloads as wl
from tests.gpu_util import DeviceWorkload, check_output, check_sets, dev, to_np
from tests.helpers import oracle_cfg, oracle_cnn
from tests.test_gpu_parity import compare_state, logit_eps

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,Hq,Hkv,D,window,budget,kernel,channels,dilation", [
    ("bf16", 4, 1, 64, 700, 333, (5,), (32,), None),                       # matrix stream, 4 shares, ragged last blocks
    ("bf16", 1, 1, 128, 500, 129, (3,), (16,), None),                      # one query head: VALU stream, 4 shares
    ("bf16", 20, 1, 64, 400, 100, (3, 3, 3), (64, 32, 16), (2, 2, 2)),     # two passes over the rows, role for stacks
    ("bf16", 3, 1, 128, 300, 70, (7,), (32,), None),                       # matrix stream at D = 128
    ("bf16", 2, 1, 128, 290, 33, (3, 3), (32, 16), (1, 3)),                # stack without a role: scored per head
    ("f32", 4, 1, 64, 300, 40, (5,), (16,), None),
    ("bf16", 4, 2, 64, 64, 20, (1,), (16,), None),                         # rho = 0: finishing launch
    ("bf16", 2, 1, 64, 40, 1 << 16, (3,), (16,), None),                    # budget of 2^16: finishing launch
])
@pytest.mark.parametrize("full", [False, True])
def test_decode_shares(dtype, Hq, Hkv, D, window, budget, kernel, channels, dilation, full):
    few = min(budget, 120)
    lens = [window + 2 * few, window + few + 5] if full else [window - 5, max(1, window // 3)]
    w = wl.make_prefill("decode_shares", 4100 + window, dtype, lens, Hq, Hkv, D, window, budget, 2, 0.0, cnn_kernel=kernel,
                        cnn_channels=channels, cnn_dilation=dilation, w_std=0.1)
    cfg, cnn = oracle_cfg(w), oracle_cnn(w.cnn)
    d = DeviceWorkload(w)
    cache = d.new_cache()
    logits = torch.empty((Hkv, w.total_tokens), dtype=torch.float32, device="cuda")
    B.ltea_prefill(d.cfg, d.cnn, d.q, d.k, d.v, d.cu, d.max_seqlen, cache, logits=logits)
    _, states, z64, _ = orc.prefill(w.q, w.k, w.v, cfg, cnn, w.cu_seqlens)
    assert not check_sets(cache, z64, w, logit_eps(to_np(logits), z64, dtype)), "pick another seed"
    ws = B.decode_workspace(d.cfg, d.cnn, w.n_seqs)
    for step in range(9):
        q, k, v = wl.decode_inputs(w.seed, step, dtype, w.n_seqs, Hq, Hkv, D)
        out = to_np(B.ltea_decode_step(d.cfg, d.cnn, dev(q, dtype), dev(k, dtype), dev(v, dtype), cache, workspace=ws))
        ref = np.stack([orc.decode_step(states[s], q[s], k[s], v[s], cfg, cnn) for s in range(w.n_seqs)])
        check_output(out, ref, dtype, f"step {step}")
        compare_state(cache, states, w, step)
