"""Eager decode steps by what scores inside them: the stack role, the single-layer role and the per-head scoring with each of its
forms (single layers of any kernel, unequal dilations, odd channel counts, weights that are not 16-byte aligned), more sequences
than a scoring workgroup takes; rotary models with either pairing, with and without unrotated keys, past their tables; and the
finishing launch of caches with more than 127 KV heads.  Oracle: the eager step, or for rotary models a lazy step and a batched
scoring after every step."""
import numpy as np
import pytest
import torch

from oracle import ltea_oracle as orc
from paper_2510_20787_amd import binding as B
from paper_2510_20787_amd import workloads as wl
from tests.gpu_util import DeviceWorkload, check_output, check_sets, dev, to_np
from tests.helpers import oracle_cfg, oracle_cnn
from tests.test_gpu_lazy import LOGIT_TOL_ROPE, compare_ring_logits_new, compare_sets
from tests.test_gpu_parity import compare_state, logit_eps

pytestmark = pytest.mark.gpu

STACK = ((3, 3, 3), (64, 32, 16), (2, 2, 2))


def prefilled(dtype, lens, Hq, Hkv, D, window, budget, cnn, w_std=0.1, seed=0):
    w = wl.make_prefill("decode_roles", 900 + seed, dtype, lens, Hq, Hkv, D, window, budget, 1, 0.0, cnn_kernel=cnn[0],
                        cnn_channels=cnn[1], cnn_dilation=cnn[2], w_std=w_std)
    d = DeviceWorkload(w)
    cache = d.new_cache()
    logits = torch.empty((Hkv, w.total_tokens), dtype=torch.float32, device="cuda")
    B.ltea_prefill(d.cfg, d.cnn, d.q, d.k, d.v, d.cu, d.max_seqlen, cache, logits=logits)
    _, states, z64, _ = orc.prefill(w.q, w.k, w.v, oracle_cfg(w), oracle_cnn(w.cnn), w.cu_seqlens)
    assert not check_sets(cache, z64, w, logit_eps(to_np(logits), z64, dtype)), "pick another seed"
    return w, d, cache, states


LENS = [70, 5, 40, 0, 90, 33, 61, 2, 50, 44]        # ten: a second, partly filled group of eight


@pytest.mark.parametrize("dtype,Hq,Hkv,D,cnn,lens", [
    ("bf16", 4, 2, 64, STACK, LENS),                                        # stack role
    ("bf16", 2, 2, 64, ((3, 3), (32, 64), (3, 3)), LENS),                   # stack role, two layers, one query head
    ("bf16", 4, 2, 64, ((3, 3, 3), (64, 32, 16), (1, 2, 4)), [80, 9]),      # unequal dilations: rows apart in every layer
    ("bf16", 4, 2, 64, ((5, 3), (32, 16), (2, 1)), [80, 9]),
    ("bf16", 2, 2, 128, ((7, 1, 3), (16, 24, 8), (2, 1, 3)), [80, 9]),      # a layer without reach in the middle
    ("bf16", 2, 1, 64, ((3, 1), (32, 16), (2, 1)), [80, 9]),                # and at the end
    ("bf16", 4, 2, 64, ((9,), (32,), (1,)), [80, 9]),                       # single layers without a role
    ("bf16", 2, 2, 128, ((5,), (48,), (3,)), [80, 9]),
    ("bf16", 4, 2, 64, ((3, 3), (20, 12), (1, 2)), [80, 9]),                # channel counts that are no runs of eight
    ("bf16", 4, 2, 64, ((3, 5), (17, 9), (1, 1)), [80, 9]),                 # nor whole pieces
    ("f32", 2, 2, 64, ((5,), (16,), (1,)), [80, 9]),
    ("f32", 4, 1, 128, ((3, 3), (19, 8), (1, 3)), [80, 9]),
    ("f32", 4, 2, 64, ((11,), (7,), (2,)), [80, 9]),
])
def test_eager_step(dtype, Hq, Hkv, D, cnn, lens):
    w, d, cache, states = prefilled(dtype, lens, Hq, Hkv, D, 48, 10, cnn, seed=len(cnn[0]) + cnn[1][0])
    cfg, ocnn = oracle_cfg(w), oracle_cnn(w.cnn)
    for step in range(7):
        q, k, v = wl.decode_inputs(w.seed, step, dtype, w.n_seqs, Hq, Hkv, D)
        out = to_np(B.ltea_decode_step(d.cfg, d.cnn, dev(q, dtype), dev(k, dtype), dev(v, dtype), cache))
        ref = np.stack([orc.decode_step(states[s], q[s], k[s], v[s], cfg, ocnn) for s in range(w.n_seqs)])
        check_output(out, ref, dtype, f"step {step}")
        compare_state(cache, states, w, step)


@pytest.mark.parametrize("dtype,cnn", [("bf16", ((9,), (32,), (1,))), ("bf16", ((3, 3, 3), (64, 32, 16), (1, 2, 4))), ("f32", ((5,), (16,), (1,)))])
def test_weights_without_alignment(dtype, cnn):
    """Weights one element past a 16-byte boundary are read element by element."""
    w, d, cache, states = prefilled(dtype, [80, 9], 4, 2, 64, 48, 10, cnn, seed=3)
    moved = []
    for l in range(len(cnn[0])):
        t = d.cnn.tensors[2 * l]
        room = torch.empty(t.numel() + 8, dtype=t.dtype, device="cuda")
        room[1:1 + t.numel()] = t.reshape(-1)
        moved.append(room)
        d.cnn.struct.w[l] = room.data_ptr() + room.element_size()
    cfg, ocnn = oracle_cfg(w), oracle_cnn(w.cnn)
    for step in range(3):
        q, k, v = wl.decode_inputs(w.seed, step, dtype, 2, 4, 2, 64)
        out = to_np(B.ltea_decode_step(d.cfg, d.cnn, dev(q, dtype), dev(k, dtype), dev(v, dtype), cache))
        ref = np.stack([orc.decode_step(states[s], q[s], k[s], v[s], cfg, ocnn) for s in range(2)])
        check_output(out, ref, dtype, f"step {step}")
        compare_state(cache, states, w, step)


@pytest.mark.parametrize("interleaved,give_k_feat,rot_dim", [(False, False, 32), (True, False, 64), (False, True, 64), (True, True, 32)])
@pytest.mark.parametrize("cnn", [STACK, ((3, 3), (64, 32), (1, 1))])
def test_rotary_stack_role(cnn, interleaved, give_k_feat, rot_dim):
    """The stack role of a rotary model, ten sequences.  With k_feat the incoming token is scored from the exact key, one rounding
    less than the oracle's procedure: its logits are compared, not its sets."""
    Hq, Hkv, D, window, budget = 4, 2, 64, 32, 8
    w = wl.make_prefill("rotary_role", 640 + rot_dim + interleaved, "bf16", LENS, Hq, Hkv, D, window, budget, 1, 0.0, cnn_kernel=cnn[0],
                        cnn_channels=cnn[1], cnn_dilation=cnn[2], w_std=0.1)
    cfg, ocnn = oracle_cfg(w), oracle_cnn(w.cnn)
    n_dec = 12
    cos, sin = wl.rope_tables(max(LENS) + n_dec + 1, rot_dim, 100.0)
    rope_o = orc.OracleRope(cos.astype(np.float64), sin.astype(np.float64), interleaved)
    rope_g = B.upload_rope(cos, sin, interleaved)
    store = lambda x: wl.to_storage(np.asarray(x, np.float32), "bf16")
    k_post = np.zeros_like(w.k)
    for s in range(w.n_seqs):
        lo, hi = int(w.cu_seqlens[s]), int(w.cu_seqlens[s + 1])
        for p in range(hi - lo):
            k_post[lo + p] = store(orc.rope_rotate(w.k[lo + p], p, rope_o))
    z64 = orc.score(w.k, w.v, ocnn, w.cu_seqlens)
    states = []
    for s in range(w.n_seqs):
        lo, hi = int(w.cu_seqlens[s]), int(w.cu_seqlens[s + 1])
        kept = [orc.retain(z64[h, lo:hi], hi - lo, window, budget, 1, 0.0) for h in range(Hkv)]
        states.append(orc.state_after_prefill(k_post[lo:hi], w.v[lo:hi], z64[:, lo:hi], cfg, w.cnn.rho, kept))
    d = DeviceWorkload(w)
    cache = d.new_cache()
    logits = torch.empty((Hkv, w.total_tokens), dtype=torch.float32, device="cuda")
    B.ltea_prefill(d.cfg, d.cnn, d.q, dev(k_post, "bf16"), d.v, d.cu, d.max_seqlen, cache, logits=logits, k_feat=d.k)
    assert not check_sets(cache, z64, w, logit_eps(to_np(logits), z64, "bf16")), "pick another seed"
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    for t in range(n_dec):
        q, k, v = wl.decode_inputs(w.seed, t, "bf16", w.n_seqs, Hq, Hkv, D)
        kp = np.stack([store(orc.rope_rotate(k[s], states[s].n_seen, rope_o)) for s in range(w.n_seqs)])
        got = to_np(B.ltea_decode_step_feat(d.cfg, d.cnn, dev(q, "bf16"), dev(kp, "bf16"), dev(v, "bf16"), cache, rope=rope_g,
                                            k_feat=dev(k, "bf16") if give_k_feat else None, status=status))
        ref = np.stack([orc.decode_step_lazy(states[s], q[s], kp[s], v[s], cfg) for s in range(w.n_seqs)])
        for st in states:
            orc.rescore(st, cfg, ocnn, rope_o, lambda x: store(x).astype(np.float64))
        check_output(got, ref, "bf16", f"step {t}")
        compare_ring_logits_new(cache, states, w, LOGIT_TOL_ROPE, z64)
        if not give_k_feat:
            compare_sets(cache, states, w, t)
    assert int(status.item()) == 0


@pytest.mark.parametrize("cnn", [STACK, ((5,), (32,), (1,)), ((3, 3), (32, 16), (1, 2))])
def test_positions_past_the_rotary_tables(cnn):
    """The status bit is set once a ring key that has to be rotated back lies past the tables, and not before; the incoming key,
    given as it was before the rotation, needs none."""
    w, d, cache, _ = prefilled("bf16", [40, 20], 4, 2, 64, 32, 8, cnn, seed=17)
    cos, sin = wl.rope_tables(42, 64, 100.0)
    rope = B.upload_rope(cos, sin, False)
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    for t, past in ((40, 0), (41, 0), (42, 0), (43, B.LTEA_ROPE_RANGE)):      # keys of positions below t come from the ring
        q, k, v = wl.decode_inputs(w.seed, t, "bf16", 2, 4, 2, 64)
        B.ltea_decode_step_feat(d.cfg, d.cnn, dev(q, "bf16"), dev(k, "bf16"), dev(v, "bf16"), cache, rope=rope, k_feat=dev(k, "bf16"),
                                status=status)
        assert int(status.item()) == past, t


@pytest.mark.parametrize("cnn", [STACK, ((5,), (32,), (1,))])
def test_more_kv_heads_than_the_counters_hold(cnn):
    w, d, cache, states = prefilled("bf16", [30], 130, 130, 64, 20, 4, cnn, seed=29)
    cfg, ocnn = oracle_cfg(w), oracle_cnn(w.cnn)
    for step in range(3):
        q, k, v = wl.decode_inputs(w.seed, step, "bf16", 1, 130, 130, 64)
        out = to_np(B.ltea_decode_step(d.cfg, d.cnn, dev(q, "bf16"), dev(k, "bf16"), dev(v, "bf16"), cache))
        check_output(out, orc.decode_step(states[0], q[0], k[0], v[0], cfg, ocnn)[None], "bf16", f"step {step}")
        compare_state(cache, states, w, step)
