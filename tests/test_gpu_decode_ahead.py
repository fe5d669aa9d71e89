"""Decode steps of grouped heads whose first rows are requested before anything is known of a sequence: every row that is not there
(ring slots past the newest token, compact slots past the count) holds NaN and must not reach an output.  Both head sizes, few and many
query heads per KV head, heads in one share, two, four and eight and more (where D = 128 requests all first rows, the ring's or none),
with and without scoring; rings just begun, partly and just filled, compact segments empty, partly and quite full.  Outputs against
fp64 attention over the rows that the cache holds after the step (the bar of test_gpu_parity)."""
import numpy as np
import pytest
import torch

from paper_2510_20787_amd import binding as B
from paper_2510_20787_amd import workloads as wl
from tests.gpu_util import OUT_TOL, dev, to_np

pytestmark = pytest.mark.gpu
Hkv, WINDOW, BUDGET, RHO = 4, 700, 330, 2


@pytest.mark.parametrize("scored", [False, True])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("n_seqs,G", [(2, 4), (16, 4), (32, 2), (65, 5), (3, 8), (33, 6)])
def test_rows_that_are_not_there(n_seqs, G, D, scored):
    Hq = G * Hkv
    rng = np.random.default_rng(n_seqs * D + G)
    cfg = B.make_cfg(Hq, Hkv, D, WINDOW, BUDGET, 0, 0.0, 0.0, "bf16")
    seen = np.array([(3, 40, 255, WINDOW - 3, WINDOW, WINDOW + 900)[i % 6] for i in range(n_seqs)], np.int32)
    cnt = np.where(seen[:, None] > WINDOW, rng.integers(0, BUDGET + 1, (n_seqs, Hkv)), 0).astype(np.int32)
    cnt[seen > WINDOW, 0], cnt[seen > WINDOW, 1] = BUDGET, 31
    draw = lambda *shape: rng.standard_normal(shape, dtype=np.float32)  # noqa: E731
    rows = {"k_win": draw(n_seqs, Hkv, WINDOW, D), "v_win": draw(n_seqs, Hkv, WINDOW, D),
            "k_ret": draw(n_seqs, Hkv, BUDGET, D), "v_ret": draw(n_seqs, Hkv, BUDGET, D)}
    z, score = draw(n_seqs, Hkv, WINDOW), np.abs(draw(n_seqs, Hkv, BUDGET)) + np.float32(1e-3)
    pos = np.broadcast_to(2 * np.arange(BUDGET, dtype=np.int32), (n_seqs, Hkv, BUDGET)).copy()
    for b in range(n_seqs):
        rows["k_win"][b, :, seen[b]:] = rows["v_win"][b, :, seen[b]:] = np.nan
        for h in range(Hkv):
            rows["k_ret"][b, h, cnt[b, h]:] = rows["v_ret"][b, h, cnt[b, h]:] = np.nan
    up = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    kw, vw, kr, vr = (dev(rows[x], "bf16") for x in ("k_win", "v_win", "k_ret", "v_ret"))
    cache = B.wrap_cache(kw, vw, up(z), kr, vr, up(score), up(pos), up(cnt), up(seen), up(np.maximum(seen - RHO, 0).astype(np.int32)))
    cnn = None
    if scored:
        c = wl.make_cnn(rng, "bf16", Hkv, D, (5,), (32,), (1,), 0.05)
        cnn = B.upload_cnn(c.kernel, c.dilation, c.w, c.bias, c.w_out, c.b_out, "bf16")
    for step in range(3):
        q, k, v = wl.decode_inputs(7, step, "bf16", n_seqs, Hq, Hkv, D)
        args = (dev(q, "bf16"), dev(k, "bf16"), dev(v, "bf16"), cache)
        out = to_np(B.ltea_decode_step(cfg, cnn, *args) if scored else B.ltea_decode_step_lazy(cfg, *args))
        now, held = cache.n_seen.cpu().numpy(), cache.ret_count.cpu().numpy()
        assert np.array_equal(now, seen + step + 1) and held.min() >= 0 and held.max() <= BUDGET
        kc, vc, krc, vrc = (to_np(x).astype(np.float64) for x in (cache.k_win, cache.v_win, cache.k_ret, cache.v_ret))
        for b in range(n_seqs):
            n = min(int(now[b]), WINDOW)
            for h in range(Hkv):
                keys = np.concatenate([kc[b, h, :n], krc[b, h, :held[b, h]]])
                vals = np.concatenate([vc[b, h, :n], vrc[b, h, :held[b, h]]])
                s = keys @ q[b, h * G:(h + 1) * G].astype(np.float64).T * D ** -0.5
                p = np.exp(s - s.max(axis=0))
                ref = (p / p.sum(axis=0)).T @ vals
                assert np.abs(out[b, h * G:(h + 1) * G] - ref).max() <= OUT_TOL["bf16"], (step, b, h)
