"""Where the token leaving the window goes, over compact segments at and beside the number of entries that the step's threads hold
before they know whether they need them (two per thread of 4 or 8 waves), full and filling, ties at the lowest key; one, four and
eight query heads per KV head, one workgroup and several shares per head.  Kept sets: the oracle's rule replayed on the same logits.
Outputs: fp64 attention over the rows that the cache holds after the step (bf16 storage: the bar of test_gpu_parity)."""
import numpy as np
import pytest
import torch

from oracle import ltea_oracle as orc
from paper_2510_20787_amd import binding as B
from paper_2510_20787_amd import workloads as wl
from tests.gpu_util import OUT_TOL, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_seqs,Hq,Hkv,D,window,budget,missing", [
    (1, 4, 1, 64, 33, 1, 0),
    (2, 4, 1, 64, 96, 511, 2),
    (3, 8, 2, 64, 100, 512, 0),
    (260, 4, 2, 64, 40, 513, 0),         # four waves per workgroup: threads hold 512 entries
    (2, 2, 2, 128, 64, 1023, 1),
    (3, 2, 2, 64, 48, 1025, 0),
    (2, 8, 1, 128, 70, 2100, 3),
])
def test_eviction(n_seqs, Hq, Hkv, D, window, budget, missing):
    st = wl.make_decode_state("eviction", 77 + budget, "bf16", n_seqs, Hq, Hkv, D, window, budget, window + 3 * budget + 5,
                              ret_fill=budget - missing, sink=0, tau=0.0)
    rng = np.random.default_rng(budget)
    z = (rng.standard_normal((n_seqs, Hkv, window)) * 0.05).astype(np.float32)
    score = st.ret_score.copy()
    if budget > 100:                     # equal lowest keys: the latest position goes
        score[:, :, [7, budget // 2, budget - missing - 1]] = np.float32(1e-5)
    cfg = B.make_cfg(Hq, Hkv, D, window, budget, 0, 0.0, 0.0, "bf16")
    ocfg = orc.OracleCfg(Hq, Hkv, D, window, budget, 0, 0.0)
    up = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    cache = B.wrap_cache(dev(st.k_win, "bf16"), dev(st.v_win, "bf16"), up(z), dev(st.k_ret, "bf16"), dev(st.v_ret, "bf16"), up(score),
                         up(st.ret_pos), up(st.ret_count), up(st.n_seen), up(st.n_seen.copy()))
    light = [[orc.HeadState(ret_pos=[int(x) for x in st.ret_pos[b, h, :st.ret_count[b, h]]],
                            ret_key=[np.float32(x) for x in score[b, h, :st.ret_count[b, h]]],
                            ret_k=[None] * int(st.ret_count[b, h]), ret_v=[None] * int(st.ret_count[b, h]))
              for h in range(Hkv)] for b in range(n_seqs)]
    n0 = int(st.n_seen[0])
    for step in range(6):
        q, k, v = wl.decode_inputs(5, step, "bf16", n_seqs, Hq, Hkv, D)
        out = B.ltea_decode_step_lazy(cfg, dev(q, "bf16"), dev(k, "bf16"), dev(v, "bf16"), cache).float().cpu().numpy()
        e = n0 + step - window
        for b in range(n_seqs):
            for h in range(Hkv):
                orc.evict_into_retained(light[b][h], e, float(z[b, h, (n0 + step) % window]), None, None, ocfg)
        pos, cnt = cache.ret_pos.cpu().numpy(), cache.ret_count.cpu().numpy()
        kw, vw, kr, vr = (x.float().cpu().numpy().astype(np.float64) for x in (cache.k_win, cache.v_win, cache.k_ret, cache.v_ret))
        assert np.all(cache.n_seen.cpu().numpy() == n0 + step + 1)
        for b in range(n_seqs):
            for h in range(Hkv):
                n = int(cnt[b, h])
                np.testing.assert_array_equal(np.sort(pos[b, h, :n]), np.sort(light[b][h].ret_pos), err_msg=f"step {step} sequence {b} head {h}")
                keys, vals = np.concatenate([kw[b, h], kr[b, h, :n]]), np.concatenate([vw[b, h], vr[b, h, :n]])
                np.testing.assert_array_equal(keys[(n0 + step) % window], k[b, h])
                for g in range(Hq // Hkv):
                    hq = h * (Hq // Hkv) + g
                    s = keys @ q[b, hq].astype(np.float64) * D ** -0.5
                    p = np.exp(s - s.max())
                    assert np.abs(out[b, hq] - p @ vals / p.sum()).max() <= OUT_TOL["bf16"]
