"""Lazy decode steps of grouped heads while the ring is filling: its rows are requested before the number of tokens is known, so
what unused slots hold (here NaN) must not reach an output.  Rings that end inside a block of 32 slots, the incoming token in
the first and the last slot of a block, few (terms as columns) and many query heads, both head sizes; and full rings, where
the incoming token replaces the evicted row.  Outputs and retained sets against the oracle."""
import numpy as np
import pytest
import torch

from oracle import ltea_oracle as orc
from paper_2510_20787_amd import binding as B
from paper_2510_20787_amd import workloads as wl
from tests.gpu_util import DeviceWorkload, check_output, check_sets, dev, to_np
from tests.helpers import oracle_cfg, oracle_cnn
from tests.test_gpu_lazy import compare_sets
from tests.test_gpu_parity import logit_eps

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,D,window,budget", [
    (4, 1, 64, 300, 33), (5, 1, 64, 64, 20), (8, 1, 64, 130, 40), (3, 1, 128, 95, 31), (12, 2, 128, 257, 64)])
@pytest.mark.parametrize("lens", ["short", "full"])
def test_lazy_step_while_the_ring_fills(Hq, Hkv, D, window, budget, lens):
    lens = [30, 60, window - 4] if lens == "short" else [window + 2 * budget + 40, window + 31, window]
    w = wl.make_prefill("lazy_ring", 6100 + window, "bf16", lens, Hq, Hkv, D, window, budget, 2, 0.0, cnn_kernel=(5,),
                        cnn_channels=(32,), w_std=0.1)
    cfg, cnn = oracle_cfg(w), oracle_cnn(w.cnn)
    d = DeviceWorkload(w)
    cache = d.new_cache()
    logits = torch.empty((Hkv, w.total_tokens), dtype=torch.float32, device="cuda")
    B.ltea_prefill(d.cfg, d.cnn, d.q, d.k, d.v, d.cu, d.max_seqlen, cache, logits=logits)
    _, states, z64, _ = orc.prefill(w.q, w.k, w.v, cfg, cnn, w.cu_seqlens)
    assert not check_sets(cache, z64, w, logit_eps(to_np(logits), z64, "bf16")), "pick another seed"
    for s, n in enumerate(lens):
        cache.k_win[s, :, n:] = float("nan")
        cache.v_win[s, :, n:] = float("nan")
    for step in range(7):
        q, k, v = wl.decode_inputs(w.seed, step, "bf16", w.n_seqs, Hq, Hkv, D)
        out = to_np(B.ltea_decode_step_lazy(d.cfg, dev(q, "bf16"), dev(k, "bf16"), dev(v, "bf16"), cache))
        ref = np.stack([orc.decode_step(states[s], q[s], k[s], v[s], cfg, cnn) for s in range(w.n_seqs)])
        check_output(out, ref, "bf16", f"step {step}")
        compare_sets(cache, states, w, step)
