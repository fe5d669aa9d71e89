"""GPU parity of ltea_prefill_append: continuing a prefill on an existing cache state must give the rows and
the final state of one oracle prefill over the whole history (the kept set is nested in the prefix length, so
re-selecting among the old kept entries and the tokens that leave the window now is the same as selecting among
everything).  The history is cut at several points: inside the window, exactly at it, far beyond it, in more than
one chunk, after decode steps (compact segment no longer ordered), with empty chunks for some sequences."""
import numpy as np
import pytest
import torch

from oracle import ltea_oracle as orc
from paper_2510_20787_amd import binding as B
from paper_2510_20787_amd import workloads as wl
from tests.gpu_util import LOGIT_TOL, OUT_TOL, check_sets, dev, to_np
from tests.helpers import oracle_cfg, oracle_cnn

pytestmark = pytest.mark.gpu


def pack(x, cu, cuts_lo, cuts_hi):
    """Rows [cuts_lo[s], cuts_hi[s]) of every sequence, packed."""
    parts = [x[int(cu[s]) + cuts_lo[s]: int(cu[s]) + cuts_hi[s]] for s in range(len(cu) - 1)]
    return np.ascontiguousarray(np.concatenate(parts, axis=0)) if parts else x[:0]


def cu_of(lens):
    cu = np.zeros(len(lens) + 1, dtype=np.int32)
    cu[1:] = np.cumsum(lens)
    return cu


CASES = {
    # name: (seqlens, Hq, Hkv, D, window, budget, sink, tau, kernel, channels, dilation, list of cut fractions)
    "d64": ([700, 129, 300, 40], 4, 2, 64, 96, 40, 0, 0.0, (5,), (32,), None, [0.5]),
    "d64_chunks": ([900, 257], 4, 4, 64, 64, 24, 2, 0.0, (5,), (32,), None, [0.2, 0.55, 0.8]),
    "d128_gqa_sink": ([513, 391, 70], 8, 2, 128, 128, 48, 4, 0.0, (7,), (32,), None, [0.6]),
    "d64_deep": ([600, 333], 8, 2, 64, 96, 40, 4, 0.0, (3, 3, 3), (64, 32, 16), (2, 2, 2), [0.1, 0.7]),
    "d64_topb": ([640], 2, 2, 64, 64, 33, 0, -np.inf, (5,), (32,), None, [0.3, 0.31]),
    "d64_budget0": ([300, 200], 2, 2, 64, 64, 0, 3, 0.0, (5,), (16,), None, [0.5]),
    # a chunk of 33 on one head per workgroup: two of the four waves have no row, and all kept entries lie in their past
    "d64_chunk33": ([400], 4, 4, 64, 64, 96, 0, -np.inf, (5,), (32,), None, [367 / 400]),
    "d128_chunk33": ([433], 2, 2, 128, 96, 130, 0, -np.inf, (5,), (32,), None, [400 / 433]),
}


def make(name):
    lens, Hq, Hkv, D, w, b, s, tau, ker, ch, dil, cuts = CASES[name]
    work = wl.make_prefill(name, 7000 + sum(map(ord, name)), "bf16", lens, Hq, Hkv, D, w, b, s, tau,
                           cnn_kernel=ker, cnn_channels=ch, cnn_dilation=dil, qkv_scale=1.0, w_std=0.05)
    return work, cuts


def device_setup(w):
    cfg = B.make_cfg(w.Hq, w.Hkv, w.D, w.window, w.budget, w.sink, w.tau, 0.0, w.dtype)
    c = w.cnn
    cnn = B.upload_cnn(c.kernel, c.dilation, c.w, c.bias, c.w_out, c.b_out, w.dtype)
    return cfg, cnn


def check_final_state(w, cache, ref_states, z64, eps, logit_tol=LOGIT_TOL["bf16"]):
    near = check_sets(cache, z64, w, eps)
    assert len(near) <= max(1, w.n_seqs // 64), f"heads inside the decision margin: {near}"
    rho = w.cnn.rho
    kw, vw, zw = to_np(cache.k_win), to_np(cache.v_win), to_np(cache.win_score)
    kr, vr = to_np(cache.k_ret), to_np(cache.v_ret)
    cnts, poss = cache.ret_count.cpu().numpy(), cache.ret_pos.cpu().numpy()
    n_seen, n_scored = cache.n_seen.cpu().numpy(), cache.n_scored.cpu().numpy()
    for s in range(w.n_seqs):
        lo, hi = int(w.cu_seqlens[s]), int(w.cu_seqlens[s + 1])
        n = hi - lo
        assert int(n_seen[s]) == n and int(n_scored[s]) == max(0, n - rho)
        for h in range(w.Hkv):
            # ring rows of every valid position, their final logits, and the kept rows
            for p in range(max(0, n - w.window), n):
                slot = p % w.window
                np.testing.assert_array_equal(kw[s, h, slot], w.k[lo + p, h])
                np.testing.assert_array_equal(vw[s, h, slot], w.v[lo + p, h])
            for p in range(max(0, n - w.window), max(0, n - rho)):
                ref = z64[h, lo + p]
                assert abs(float(zw[s, h, p % w.window]) - ref) <= logit_tol * max(1.0, abs(ref))
            for r in range(int(cnts[s, h])):
                np.testing.assert_array_equal(kr[s, h, r], w.k[lo + poss[s, h, r], h])
                np.testing.assert_array_equal(vr[s, h, r], w.v[lo + poss[s, h, r], h])
    return set(near)


@pytest.mark.parametrize("name", list(CASES))
def test_append_equals_one_shot_prefill(name):
    w, fracs = make(name)
    ocfg, ocnn = oracle_cfg(w), oracle_cnn(w.cnn)
    ref_out, ref_states, z64, kept = orc.prefill(w.q, w.k, w.v, ocfg, ocnn, w.cu_seqlens)
    cfg, cnn = device_setup(w)
    cu = w.cu_seqlens
    lens = [int(cu[s + 1] - cu[s]) for s in range(w.n_seqs)]
    # cut points per sequence; the second sequence gets an empty chunk somewhere to exercise M = 0
    cuts = [[0] * w.n_seqs]
    for f in fracs:
        cuts.append([min(lens[s], int(round(f * lens[s]))) for s in range(w.n_seqs)])
    cuts.append(lens)
    if w.n_seqs > 1 and len(cuts) > 2:
        cuts[-2][1] = cuts[-1][1]          # sequence 1 is complete one chunk early: its last chunk is empty
    cache = B.alloc_cache(cfg, w.n_seqs)
    got = np.zeros_like(ref_out, dtype=np.float32)
    for c in range(len(cuts) - 1):
        a, b = cuts[c], cuts[c + 1]
        m = [b[s] - a[s] for s in range(w.n_seqs)]
        q, k, v = (dev(pack(x, cu, a, b), w.dtype) for x in (w.q, w.k, w.v))
        cu_c = torch.from_numpy(cu_of(m)).cuda()
        if c == 0:
            out = B.ltea_prefill(cfg, cnn, q, k, v, cu_c, max(max(m), 1), cache)
        else:
            out = B.ltea_prefill_append(cfg, cnn, q, k, v, cu_c, max(max(m), 1), cache)
        o = to_np(out)
        off = 0
        for s in range(w.n_seqs):
            if c > 0:     # rows of the first chunk saw the first chunk's kept set, not the final one
                got[int(cu[s]) + a[s]: int(cu[s]) + b[s]] = o[off: off + m[s]]
            off += m[s]
    torch.cuda.synchronize()
    skip = check_final_state(w, cache, ref_states, z64, 1e-5)
    # appended rows of the LAST chunk saw the final kept set: they must equal the one-shot rows
    G = w.Hq // w.Hkv
    a = cuts[-2]
    worst, scale = 0.0, 0.0
    for s in range(w.n_seqs):
        lo = int(cu[s])
        for hq in range(w.Hq):
            if (s, hq // G) in skip:
                continue
            rows = slice(lo + a[s], lo + lens[s])
            if a[s] == lens[s]:
                continue
            worst = max(worst, float(np.abs(got[rows, hq] - ref_out[rows, hq]).max()))
            scale = max(scale, float(np.abs(ref_out[rows, hq]).max()))
    assert worst <= OUT_TOL["bf16"] and worst <= OUT_TOL["bf16"] * scale, (worst, scale)


def test_append_after_decode_steps():
    """Prefill, a run of decode steps (the compact segment is then no longer ordered by position: replacements
    happen in place), then a continuation: state and appended rows must still equal the one-shot prefill."""
    lens = [520, 410]
    w = wl.make_prefill("append_after_decode", 7777, "bf16", lens, 4, 2, 64, 64, 20, 1, 0.0,
                        cnn_kernel=(5,), cnn_channels=(32,), qkv_scale=1.0, w_std=0.05)
    ocfg, ocnn = oracle_cfg(w), oracle_cnn(w.cnn)
    ref_out, ref_states, z64, kept = orc.prefill(w.q, w.k, w.v, ocfg, ocnn, w.cu_seqlens)
    cfg, cnn = device_setup(w)
    cu = w.cu_seqlens
    n_pre, n_dec = [300, 200], 90
    cache = B.alloc_cache(cfg, w.n_seqs)
    zero = [0, 0]
    q, k, v = (dev(pack(x, cu, zero, n_pre), w.dtype) for x in (w.q, w.k, w.v))
    B.ltea_prefill(cfg, cnn, q, k, v, torch.from_numpy(cu_of(n_pre)).cuda(), max(n_pre), cache)
    for t in range(n_dec):
        idx = [int(cu[s]) + n_pre[s] + t for s in range(w.n_seqs)]
        B.ltea_decode_step(cfg, cnn, dev(w.q[idx], w.dtype), dev(w.k[idx], w.dtype), dev(w.v[idx], w.dtype), cache)
    a = [n_pre[s] + n_dec for s in range(w.n_seqs)]
    m = [lens[s] - a[s] for s in range(w.n_seqs)]
    q, k, v = (dev(pack(x, cu, a, lens), w.dtype) for x in (w.q, w.k, w.v))
    out = to_np(B.ltea_prefill_append(cfg, cnn, q, k, v, torch.from_numpy(cu_of(m)).cuda(), max(m), cache))
    torch.cuda.synchronize()
    skip = check_final_state(w, cache, ref_states, z64, 1e-5)
    G = w.Hq // w.Hkv
    off, worst = 0, 0.0
    for s in range(w.n_seqs):
        rows = slice(int(cu[s]) + a[s], int(cu[s]) + lens[s])
        for hq in range(w.Hq):
            if (s, hq // G) not in skip:
                worst = max(worst, float(np.abs(out[off: off + m[s], hq] - ref_out[rows, hq]).max()))
        off += m[s]
    assert worst <= OUT_TOL["bf16"], worst


def test_append_many_sequences():
    """300 sequences (the planning kernel walks them 256 at a time; the sequence lookup 64 at a time), random
    cut points including empty first or second parts."""
    rng = np.random.default_rng(99)
    lens = [int(x) for x in rng.integers(1, 160, size=300)]
    w = wl.make_prefill("append_many", 9090, "bf16", lens, 2, 2, 64, 48, 10, 1, 0.0, cnn_kernel=(5,), cnn_channels=(32,),
                        qkv_scale=1.0, w_std=0.05)
    ocfg, ocnn = oracle_cfg(w), oracle_cnn(w.cnn)
    ref_out, ref_states, z64, kept = orc.prefill(w.q, w.k, w.v, ocfg, ocnn, w.cu_seqlens)
    cfg, cnn = device_setup(w)
    cu = w.cu_seqlens
    cut = [int(rng.integers(0, n + 1)) for n in lens]
    zero = [0] * w.n_seqs
    cache = B.alloc_cache(cfg, w.n_seqs)
    q, k, v = (dev(pack(x, cu, zero, cut), w.dtype) for x in (w.q, w.k, w.v))
    B.ltea_prefill(cfg, cnn, q, k, v, torch.from_numpy(cu_of(cut)).cuda(), max(max(cut), 1), cache)
    m = [lens[s] - cut[s] for s in range(w.n_seqs)]
    q, k, v = (dev(pack(x, cu, cut, lens), w.dtype) for x in (w.q, w.k, w.v))
    out = to_np(B.ltea_prefill_append(cfg, cnn, q, k, v, torch.from_numpy(cu_of(m)).cuda(), max(max(m), 1), cache))
    torch.cuda.synchronize()
    skip = check_final_state(w, cache, ref_states, z64, 1e-5)
    off, worst = 0, 0.0
    for s in range(w.n_seqs):
        rows = slice(int(cu[s]) + cut[s], int(cu[s]) + lens[s])
        for hq in range(w.Hq):
            if m[s] and (s, hq) not in skip:
                worst = max(worst, float(np.abs(out[off: off + m[s], hq] - ref_out[rows, hq]).max()))
        off += m[s]
    assert worst <= OUT_TOL["bf16"], worst


@pytest.mark.parametrize("n_first", [0, 1, 5, 11])
def test_append_to_a_history_shorter_than_the_receptive_field(n_first):
    """Multi-layer CNN and a first chunk of at most 2 rho tokens (or none at all): the continuation must score the
    positions next to the sequence start with real zero padding at every layer, not with the activations of zero
    input rows standing in front of the ring."""
    lens = [150, 90]
    w = wl.make_prefill("append_short_history", 7100 + n_first, "bf16", lens, 4, 2, 64, 64, 12, 2, 0.0,
                        cnn_kernel=(3, 3, 3), cnn_channels=(64, 32, 16), cnn_dilation=(2, 2, 2), qkv_scale=1.0, w_std=0.05)
    ocfg, ocnn = oracle_cfg(w), oracle_cnn(w.cnn)
    ref_out, ref_states, z64, kept = orc.prefill(w.q, w.k, w.v, ocfg, ocnn, w.cu_seqlens)
    cfg, cnn = device_setup(w)
    cu = w.cu_seqlens
    cache = B.alloc_cache(cfg, w.n_seqs)
    a = [n_first, min(n_first, 3)]
    zero = [0, 0]
    if n_first > 0:
        q, k, v = (dev(pack(x, cu, zero, a), w.dtype) for x in (w.q, w.k, w.v))
        B.ltea_prefill(cfg, cnn, q, k, v, torch.from_numpy(cu_of(a)).cuda(), max(a), cache)
    else:
        a = zero
    m = [lens[s] - a[s] for s in range(w.n_seqs)]
    q, k, v = (dev(pack(x, cu, a, lens), w.dtype) for x in (w.q, w.k, w.v))
    out = to_np(B.ltea_prefill_append(cfg, cnn, q, k, v, torch.from_numpy(cu_of(m)).cuda(), max(m), cache))
    skip = check_final_state(w, cache, ref_states, z64, 1e-5)
    G = w.Hq // w.Hkv
    off = 0
    for s in range(w.n_seqs):
        rows = slice(int(cu[s]) + a[s], int(cu[s]) + lens[s])
        for hq in range(w.Hq):
            if (s, hq // G) not in skip:
                err = float(np.abs(out[off: off + m[s], hq] - ref_out[rows, hq]).max())
                assert err <= OUT_TOL["bf16"] * float(np.abs(ref_out[rows, hq]).max()), (s, hq, err)
        off += m[s]


@pytest.mark.parametrize("interleaved,give_k_feat,rot_dim", [(False, True, 64), (True, False, 64), (False, False, 32)])
def test_append_for_a_rotary_model(interleaved, give_k_feat, rot_dim):
    """Rotary models cache rotated keys and score unrotated ones.  First chunk: ltea_prefill with k_feat.  Second chunk:
    ltea_prefill_append_feat with the model's tables; the ring is rotated back for the scoring, the new keys come
    unrotated from the caller or are rotated back as well.  Oracle: one prefill over the whole history whose logits
    come from the same keys the device scored (exact ones where the first call scored them, rotated-back and rounded
    ones afterwards), everything else from the rotated keys."""
    lens, Hq, Hkv, D, window, budget, sink = [420, 260, 90], 4, 2, 64, 64, 24, 2
    w = wl.make_prefill("append_rotary", 8800 + rot_dim + int(interleaved), "bf16", lens, Hq, Hkv, D, window, budget, sink,
                        0.0, cnn_kernel=(3, 3), cnn_channels=(32, 16), cnn_dilation=(2, 1), w_std=0.1)
    # ring full / full / still filling (the sequence start is in the ring)
    near = rotary_append_run(w, [200, 100, 30], rot_dim, interleaved, give_k_feat)
    assert len(near) <= 1, near


def rotary_append_run(w, cut, rot_dim, interleaved, give_k_feat):
    """Prefill of the first cut[s] tokens with k_feat, continuation with the tables; returns the heads whose kept set
    sits inside the decision margin (everything else is asserted)."""
    import dataclasses
    dt = w.dtype
    lens = [int(w.cu_seqlens[s + 1] - w.cu_seqlens[s]) for s in range(w.n_seqs)]
    Hq, Hkv, D, window, budget, sink = w.Hq, w.Hkv, w.D, w.window, w.budget, w.sink
    ocfg, ocnn = oracle_cfg(w), oracle_cnn(w.cnn)
    rho = w.cnn.rho
    cos, sin = wl.rope_tables(max(lens) + 1, rot_dim, 100.0)
    rope_o = orc.OracleRope(cos.astype(np.float64), sin.astype(np.float64), interleaved)
    rope_g = B.upload_rope(cos, sin, interleaved)
    store = lambda x: wl.to_storage(np.asarray(x, np.float32), dt)
    cu = w.cu_seqlens
    k_pre = w.k
    k_post, k_back = np.zeros_like(k_pre), np.zeros_like(k_pre)
    for s in range(w.n_seqs):
        lo = int(cu[s])
        for p in range(lens[s]):
            k_post[lo + p] = store(orc.rope_rotate(k_pre[lo + p], p, rope_o))
            k_back[lo + p] = store(orc.rope_rotate(k_post[lo + p].astype(np.float64), p, rope_o, inverse=True))
    # the keys each logit was scored from
    feat_late = k_back.copy()
    if give_k_feat:
        for s in range(w.n_seqs):
            feat_late[int(cu[s]) + cut[s]: int(cu[s + 1])] = k_pre[int(cu[s]) + cut[s]: int(cu[s + 1])]
    z_first = orc.score(k_pre, w.v, ocnn, cu)
    z_late = orc.score(feat_late, w.v, ocnn, cu)
    z64 = z_late.copy()
    for s in range(w.n_seqs):
        lo = int(cu[s])
        z64[:, lo: lo + max(0, cut[s] - rho)] = z_first[:, lo: lo + max(0, cut[s] - rho)]
    wp = dataclasses.replace(w, k=k_post)
    ref_out = np.zeros((w.total_tokens, Hq, D))
    for s in range(w.n_seqs):
        lo, hi = int(cu[s]), int(cu[s + 1])
        kept = [orc.retain(z64[h, lo:hi], hi - lo, window, budget, sink, w.tau) for h in range(Hkv)]
        ref_out[lo:hi] = orc.sparse_attention_sequence(w.q[lo:hi], k_post[lo:hi], w.v[lo:hi], ocfg, kept)
    cfg, cnn = device_setup(w)
    cache = B.alloc_cache(cfg, w.n_seqs)
    zero = [0] * w.n_seqs
    q, k, v, kf = (dev(pack(x, cu, zero, cut), dt) for x in (w.q, k_post, w.v, k_pre))
    B.ltea_prefill(cfg, cnn, q, k, v, torch.from_numpy(cu_of(cut)).cuda(), max(max(cut), 1), cache, k_feat=kf)
    m = [lens[s] - cut[s] for s in range(w.n_seqs)]
    q, k, v, kf = (dev(pack(x, cu, cut, lens), dt) for x in (w.q, k_post, w.v, k_pre))
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    out = to_np(B.ltea_prefill_append(cfg, cnn, q, k, v, torch.from_numpy(cu_of(m)).cuda(), max(max(m), 1), cache,
                                      rope=rope_g, k_feat=kf if give_k_feat else None, status=status))
    assert int(status.item()) == 0
    # measured logit error of the ring, then the sets with that margin
    zw = to_np(cache.win_score)
    eps = 1e-6
    for s in range(w.n_seqs):
        lo, n = int(cu[s]), lens[s]
        for h in range(Hkv):
            for p in range(max(0, n - window), max(0, n - rho)):
                eps = max(eps, abs(float(zw[s, h, p % window]) - z64[h, lo + p]))
    assert eps <= (2e-3 if dt == "bf16" else 1e-4) * 4, eps
    skip = check_final_state_generic(wp, cache, z64, eps)
    G = Hq // Hkv
    off = 0
    scale = max(float(np.abs(ref_out).max()), 1e-30)
    for s in range(w.n_seqs):
        rows = slice(int(cu[s]) + cut[s], int(cu[s]) + lens[s])
        for hq in range(Hq):
            if m[s] and (s, hq // G) not in skip:
                err = float(np.abs(out[off: off + m[s], hq] - ref_out[rows, hq]).max())
                assert err <= OUT_TOL[dt] * max(1.0, scale), (s, hq, err)
        off += m[s]
    return skip


def check_final_state_generic(w, cache, z64, eps):
    """Counters, ring rows, kept rows and kept sets (heads inside the margin 2 * eps are returned, not compared)."""
    near = set(check_sets(cache, z64, w, eps))
    rho = w.cnn.rho
    kw, vw = to_np(cache.k_win), to_np(cache.v_win)
    kr, vr = to_np(cache.k_ret), to_np(cache.v_ret)
    cnts, poss = cache.ret_count.cpu().numpy(), cache.ret_pos.cpu().numpy()
    n_seen, n_scored = cache.n_seen.cpu().numpy(), cache.n_scored.cpu().numpy()
    for s in range(w.n_seqs):
        lo, hi = int(w.cu_seqlens[s]), int(w.cu_seqlens[s + 1])
        n = hi - lo
        assert int(n_seen[s]) == n and int(n_scored[s]) == max(0, n - rho)
        for h in range(w.Hkv):
            for p in range(max(0, n - w.window), n):
                np.testing.assert_array_equal(kw[s, h, p % w.window], w.k[lo + p, h])
                np.testing.assert_array_equal(vw[s, h, p % w.window], w.v[lo + p, h])
            for r in range(int(cnts[s, h])):
                np.testing.assert_array_equal(kr[s, h, r], w.k[lo + poss[s, h, r], h])
                np.testing.assert_array_equal(vr[s, h, r], w.v[lo + poss[s, h, r], h])
    return near


def test_append_rotary_arguments_and_table_range():
    """k_feat without tables is refused; positions beyond the tables raise the status bit and leave the call defined."""
    lens = [100]
    w = wl.make_prefill("append_rotary_args", 31, "bf16", lens, 2, 2, 64, 32, 8, 0, 0.0, cnn_kernel=(3,), cnn_channels=(16,))
    cfg, cnn = device_setup(w)
    cache = B.alloc_cache(cfg, 1)
    q, k, v = (dev(x, "bf16") for x in (w.q, w.k, w.v))
    cu1 = torch.tensor([0, 60], dtype=torch.int32, device="cuda")
    B.ltea_prefill(cfg, cnn, q[:60], k[:60], v[:60], cu1, 60, cache)
    cu2 = torch.tensor([0, 40], dtype=torch.int32, device="cuda")
    with pytest.raises(RuntimeError):
        B.ltea_prefill_append(cfg, cnn, q[60:], k[60:], v[60:], cu2, 40, cache, k_feat=k[60:])
    cos, sin = wl.rope_tables(70, 64, 100.0)              # positions 70..99 are beyond the tables
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    out = B.ltea_prefill_append(cfg, cnn, q[60:], k[60:], v[60:], cu2, 40, cache, rope=B.upload_rope(cos, sin, False),
                                status=status)
    assert int(status.item()) & B.LTEA_ROPE_RANGE
    assert int(cache.n_seen[0]) == 100 and bool(torch.isfinite(out.float()).all())


@pytest.mark.parametrize("kernel,channels,dilation", [((5,), (16,), None), ((3, 3), (16, 8), (2, 1))])
def test_append_fp32(kernel, channels, dilation):
    """fp32 storage goes through the layered scoring kernel and the one-wave-per-row attention kernel; three chunks,
    the last one of which sees the final kept set."""
    lens, Hq, Hkv, D, window, budget, sink = [260, 75, 130], 4, 2, 64, 48, 14, 2
    w = wl.make_prefill("append_f32", 4242 + len(kernel), "f32", lens, Hq, Hkv, D, window, budget, sink, 0.0,
                        cnn_kernel=kernel, cnn_channels=channels, cnn_dilation=dilation, qkv_scale=1.0, w_std=0.1)
    ocfg, ocnn = oracle_cfg(w), oracle_cnn(w.cnn)
    ref_out, ref_states, z64, kept = orc.prefill(w.q, w.k, w.v, ocfg, ocnn, w.cu_seqlens)
    cfg, cnn = device_setup(w)
    cu = w.cu_seqlens
    cuts = [[0, 0, 0], [100, 75, 20], [180, 75, 21], lens]
    cache = B.alloc_cache(cfg, w.n_seqs)
    for c in range(3):
        a, b = cuts[c], cuts[c + 1]
        m = [b[s] - a[s] for s in range(w.n_seqs)]
        q, k, v = (dev(pack(x, cu, a, b), "f32") for x in (w.q, w.k, w.v))
        cu_c = torch.from_numpy(cu_of(m)).cuda()
        if c == 0:
            B.ltea_prefill(cfg, cnn, q, k, v, cu_c, max(m), cache)
        else:
            out = to_np(B.ltea_prefill_append(cfg, cnn, q, k, v, cu_c, max(m), cache))
    near = check_sets(cache, z64, w, 1e-5)
    assert not near, near
    zw = to_np(cache.win_score)
    kw = to_np(cache.k_win)
    for s in range(w.n_seqs):
        lo, n = int(cu[s]), lens[s]
        assert int(cache.n_seen[s]) == n and int(cache.n_scored[s]) == max(0, n - w.cnn.rho)
        for h in range(Hkv):
            for p in range(max(0, n - window), n):
                np.testing.assert_array_equal(kw[s, h, p % window], w.k[lo + p, h])
            for p in range(max(0, n - window), max(0, n - w.cnn.rho)):
                assert abs(float(zw[s, h, p % window]) - z64[h, lo + p]) <= LOGIT_TOL["f32"] * max(1.0, abs(z64[h, lo + p]))
    off = 0
    a = cuts[2]
    for s in range(w.n_seqs):
        rows = slice(int(cu[s]) + a[s], int(cu[s]) + lens[s])
        m_s = lens[s] - a[s]
        if m_s:
            err = float(np.abs(out[off: off + m_s] - ref_out[rows]).max())
            assert err <= OUT_TOL["f32"] * max(1.0, float(np.abs(ref_out[rows]).max())), (s, err)
        off += m_s
