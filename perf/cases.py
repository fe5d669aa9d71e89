"""The calls whose speed matters to a user of this library, with their inputs, their unavoidable work and the
differences that another correct implementation may show.

A user is a serving engine (prefill, chunked prefill, decode) or a trainer (forward, backward, CNN backward) that calls
`paper_2510_20787_amd.binding` once per layer, with its weights, workspaces, output buffers and caches laid out
beforehand.  Head shapes, windows, budgets and CNNs are those of `workloads.py`; the lengths run from one short prompt to
its largest configuration.
"""
import ctypes
import math
import random

import torch

from paper_2510_20787_amd import binding as B

# kernel, channels and dilation of the scoring CNNs
CNNS = {"k5x16": ((5,), (16,), (1,)), "k5x32": ((5,), (32,), (1,)), "k7x32": ((7,), (32,), (1,)),
        "stack": ((3, 3, 3), (64, 32, 16), (2, 2, 2))}

# The mixer shapes: the small fp32 one, equal query and KV heads at both head sizes, the paper's grouped heads.
F32 = dict(dtype="f32", Hq=2, Hkv=2, D=64, window=64, budget=32, sink=0, cnn="k5x16")
EVEN64 = dict(dtype="bf16", Hq=16, Hkv=16, D=64, window=512, budget=256, sink=0, cnn="k5x32")
PAPER = dict(dtype="bf16", Hq=32, Hkv=8, D=64, window=768, budget=512, sink=4, cnn="stack")
WIDE = dict(dtype="bf16", Hq=16, Hkv=16, D=128, window=1024, budget=512, sink=0, cnn="k5x32")
LONG = dict(dtype="bf16", Hq=32, Hkv=32, D=128, window=2048, budget=1024, sink=0, cnn="k7x32")


def listed():
    return [
        # the smallest call: one short fp32 prompt, as in a numerics check of a model
        dict(name="prefill_f32_512", kind="prefill", B=1, n=512, ragged=0, fused=False, rope=False, **F32),
        # one chat turn of odd length on the paper's layer, rotary model (scored keys apart from cached ones)
        dict(name="prefill_one_777", kind="prefill", B=1, n=777, ragged=0, fused=False, rope=True, **PAPER),
        # an ordinary batch of prompts, plain multi-head layer
        dict(name="prefill_even64_4x4096", kind="prefill", B=4, n=4096, ragged=0, fused=False, rope=False, **EVEN64),
        # the same batch on the paper's layer (grouped heads, three-layer CNN)
        dict(name="prefill_paper_4x4096", kind="prefill", B=4, n=4096, ragged=0, fused=False, rope=False, **PAPER),
        # prompts of a busy server packed without padding, q, k, v views of one projection's output
        dict(name="prefill_ragged_16x16384", kind="prefill", B=16, n=16384, ragged=4, fused=True, rope=False, **WIDE),
        # one whole document
        dict(name="prefill_long_32768", kind="prefill", B=1, n=32768, ragged=0, fused=False, rope=False, **LONG),
        # one chunk of a chunked prefill: 384 more tokens on four running sequences
        dict(name="append_4x384", kind="append", B=4, n=384, hist=3000, ragged=0, fused=False, **PAPER),
        # interactive decode: one sequence, the step that neither allocates nor takes a workspace
        dict(name="decode_one", kind="decode", B=1, static=True, rope=False, **PAPER),
        # batched decode of a rotary model
        dict(name="decode_rope_32", kind="decode", B=32, static=False, rope=True, **PAPER),
        # batched decode, 800 MB of cache read per step
        dict(name="decode_wide_64", kind="decode", B=64, static=False, rope=False, **WIDE),
        # lazy scoring: a whole period of steps that do not score and the one batched scoring they need
        dict(name="decode_lazy_32", kind="lazy", B=32, **PAPER),
        # one training step's share of this layer: forward, attention backward, CNN backward
        dict(name="train_paper_4x4096", kind="train", B=4, n=4096, ragged=0, fused=False, **PAPER),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _cost(case):
    w = work(case)
    return max(w["bytes"], w["flops"] / 50)


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["prefill"] * 5 + ["decode"] * 3 + ["append"] * 2 + ["train"] * 2 + ["lazy"])
        shape = dict(rng.choice({"train": [PAPER, EVEN64, WIDE], "lazy": [PAPER, EVEN64, WIDE]}.get(
            kind, [F32, EVEN64, EVEN64, PAPER, PAPER, PAPER, WIDE, WIDE, LONG])))
        if rng.random() < 0.4:      # windows and budgets other than the tuned ones
            shape["window"] = rng.randint(shape["window"] // 2, shape["window"])
            shape["budget"] = rng.randint(shape["budget"] // 2, shape["budget"])
        case = dict(kind=kind, **shape)
        if kind in ("prefill", "append", "train"):
            total = _log_int(rng, 128, {"f32": 2048}.get(shape["dtype"], 16384 if kind == "train" else 131072))
            case["B"] = min(_log_int(rng, 1, 16), total // 64)
            case["n"] = total // case["B"]
            case["ragged"] = rng.randint(1, 1 << 20) if case["B"] > 1 and rng.random() < 0.5 else 0
            case["fused"] = rng.random() < 0.4
            if kind == "prefill":
                case["rope"] = not case["fused"] and rng.random() < 0.3
            if kind == "append":
                case["n"] = min(case["n"], 4096)
                case["hist"] = _log_int(rng, 64, 1024 if shape["dtype"] == "f32" else 8192)
        else:
            case["B"] = _log_int(rng, 1, 32 if kind == "lazy" else 128)
            if kind == "decode":
                case["rope"] = rng.random() < 0.3
                case["static"] = not case["rope"] and case["B"] <= 8 and rng.random() < 0.5
        if _cost(case) <= most:
            return case


# ---------------------------------------------------------------------------------------------------------------------
def _lengths(case):
    """Tokens per sequence of a packed batch."""
    if not case["ragged"]:
        return [case["n"]] * case["B"]
    r = random.Random(case["ragged"])
    return [r.randint(max(16, case["n"] // 16), case["n"]) for _ in range(case["B"])]


def _shares(case):
    """Share of the tokens that each KV head's threshold lets through: from a quarter of what fills the budget to four
    times as much, so that some heads stay below their cap and some overflow it, as in a trained model.  A trainer's
    heads all keep what the cap will allow later."""
    n = case.get("hist", 0) + case["n"]
    full = case["budget"] / max(n, 2 * case["budget"])
    if case["kind"] == "train":
        return [full] * case["Hkv"]
    return [min(0.9, full * 2.0 ** (-2 + 4 * (h + 0.5) / case["Hkv"])) for h in range(case["Hkv"])]


def _pairs(case):
    """(query, key) pairs that one query head of every KV head sees, summed over KV heads and sequences."""
    total, w, past = 0.0, case["window"], case.get("hist", 0)
    for n in _lengths(case):
        end = past + n
        out = max(0, end - w)
        band = sum(min(i + 1, w) for i in range(past, end))
        for share in _shares(case):
            kept = share * out if case["kind"] == "train" else min(case["budget"], share * out)
            seen = out * kept / 2 if past == 0 else n * kept * (1 - n / (2 * max(out, n)))
            total += band + seen
    return total


def _cnn_macs(case):
    """Multiply-adds of one token and KV head, and the weights of one KV head."""
    kernel, channels, _ = CNNS[case["cnn"]]
    macs, c_in = 0, 2 * case["D"]
    for k, c in zip(kernel, channels):
        macs += k * c_in * c
        c_in = c
    return macs + c_in


def work(case):
    size = 4 if case["dtype"] == "f32" else 2
    Hq, Hkv, D, w, b = (case[x] for x in ("Hq", "Hkv", "D", "window", "budget"))
    row, weights = 2 * D * size, Hkv * _cnn_macs(case) * size
    if case["kind"] in ("decode", "lazy"):
        steps = w - 2 * _rho(case) if case["kind"] == "lazy" else 1
        scored = steps * case["B"] * Hkv
        per_step = case["B"] * (Hkv * (w + b) * row + Hkv * row * 2 + 2 * Hq * D * size)
        nbytes = steps * per_step + weights + (case["B"] * Hkv * w * row if case["kind"] == "lazy" else 0)
        flops = steps * case["B"] * Hq * (w + b) * 4 * D + scored * 2 * _cnn_macs(case)
        return {"bytes": nbytes, "flops": flops}
    lens = _lengths(case)
    total = sum(lens)
    pairs = _pairs(case) * (Hq // Hkv)
    qkvo = total * (2 * Hq * D * size + Hkv * row)
    if case["kind"] == "train":
        # forward 4 D per pair, backward 10 D; the CNN once forward and twice back; gradients of q, k, v and of the
        # scored keys and values written, out and dout read
        nbytes = 2 * qkvo + total * (2 * Hq * D * size + 2 * Hkv * row) + 4 * total * (2 * Hkv + Hq) + 3 * weights
        return {"bytes": nbytes, "flops": pairs * 14 * D + 6.0 * total * Hkv * _cnn_macs(case)}
    kept_rows = 0
    for n in lens:
        end = case.get("hist", 0) + n
        new_window = min(w, n)
        kept_rows += Hkv * new_window + sum(min(b, s * max(0, end - w)) for s in _shares(case))
    nbytes = qkvo + weights + kept_rows * row
    if case["kind"] == "append":
        nbytes += len(lens) * Hkv * min(w + b, case["hist"]) * row
    if case.get("rope"):
        nbytes += total * Hkv * D * size
    return {"bytes": nbytes, "flops": pairs * 4 * D + 2.0 * total * Hkv * _cnn_macs(case)}


def tolerance(case):
    # bf16: P and O are rounded to 8 bits; fp32: sums of some hundred terms.  A near tie of two fp32 logits at the
    # threshold or at the cap may fall either way.
    return {"rel": 1e-5, "differ": 1e-3} if case["dtype"] == "f32" else {"rel": 1e-2, "differ": 1e-3}


# ---------------------------------------------------------------------------------------------------------------------
def _rho(case):
    kernel, _, dilation = CNNS[case["cnn"]]
    return sum(d * (k - 1) // 2 for k, d in zip(kernel, dilation))


def _normal(g, *shape, dtype=torch.float32, scale=1.0):
    x = torch.randn(shape, generator=g, device="cuda", dtype=dtype)
    return x if scale == 1.0 else x * scale


def _cnn(case, g, cfg, k=None, v=None, cu=None, longest=0):
    """Random weights as in `workloads.make_cnn`; with k, v given, output biases such that every head's threshold lets
    its share of these tokens through (a grid of 2^-12 keeps them independent of the last bits of the logits)."""
    kernel, channels, dilation = CNNS[case["cnn"]]
    std, c_in, ws, bs = 0.1 if case["dtype"] == "f32" else 0.05, 2 * case["D"], [], []
    for kk, c in zip(kernel, channels):
        ws.append(_normal(g, case["Hkv"], c, c_in, kk) * std)
        bs.append(_normal(g, case["Hkv"], c) * std)
        c_in = c
    w_out, b_out = _normal(g, case["Hkv"], c_in) * std, torch.zeros(case["Hkv"], device="cuda")
    make = lambda bias: B.upload_cnn(kernel, dilation, ws, bs, w_out, bias, case["dtype"])  # noqa: E731
    cnn = make(b_out)
    if k is not None:
        z = B.ltea_score(cfg, cnn, k, v, cu, longest)
        for h, share in enumerate(_shares(case)):
            at = max(1, min(z.shape[1], int(round((1 - share) * z.shape[1]))))
            b_out[h] = -z[h].kthvalue(at).values
        cnn = make(torch.round(b_out * 4096) / 4096)
    return cnn if case["kind"] == "train" else B.prepare_cnn(cfg, cnn)


def _qkv(case, g, total):
    dt = B.torch_dtype(case["dtype"])
    Hq, Hkv, D = case["Hq"], case["Hkv"], case["D"]
    scale = D ** -0.5 if case["D"] == 64 and Hq == Hkv and dt == torch.bfloat16 else 1.0
    if case["fused"]:
        return _normal(g, total, Hq + 2 * Hkv, D, dtype=dt, scale=scale).split([Hq, Hkv, Hkv], dim=1)
    return tuple(_normal(g, total, h, D, dtype=dt, scale=scale) for h in (Hq, Hkv, Hkv))


def _cu(lens):
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    return torch.tensor(cu, dtype=torch.int32, device="cuda")


def _running_cache(case, g, cfg):
    """Caches of B sequences in mid-generation: a full ring and a full compact segment each, of their own lengths."""
    Bn, Hkv, w, b, D = case["B"], case["Hkv"], case["window"], case["budget"], case["D"]
    dt, rho = B.torch_dtype(case["dtype"]), _rho(case)
    seen = w + 2 * b + torch.randint(0, 8192, (Bn,), generator=g, device="cuda", dtype=torch.int32)
    left = (seen - w).view(Bn, 1, 1).float()
    step = torch.rand((Bn, Hkv, b), generator=g, device="cuda") + torch.arange(b, device="cuda")
    pos = torch.minimum((step * left / b).floor(), left - 1).to(torch.int32)
    score = _normal(g, Bn, Hkv, b).abs() * 0.05 + 1e-6
    score[pos < case["sink"]] = float("inf")
    return B.wrap_cache(_normal(g, Bn, Hkv, w, D, dtype=dt), _normal(g, Bn, Hkv, w, D, dtype=dt), _normal(g, Bn, Hkv, w) * 0.05,
                        _normal(g, Bn, Hkv, b, D, dtype=dt), _normal(g, Bn, Hkv, b, D, dtype=dt), score, pos,
                        torch.full((Bn, Hkv), b, dtype=torch.int32, device="cuda"), seen, seen - rho)


def _cache_tensors(c):
    return [c.k_win, c.v_win, c.win_score, c.k_ret, c.v_ret, c.ret_score, c.ret_pos, c.ret_count, c.n_seen, c.n_scored]


def _bytes(n):
    return torch.empty(max(int(n), 16), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    s = {"kind": case["kind"], "case": case}
    cfg = s["cfg"] = B.make_cfg(case["Hq"], case["Hkv"], case["D"], case["window"], case["budget"], case["sink"],
                                dtype=case["dtype"])
    dt = B.torch_dtype(case["dtype"])
    if case["kind"] in ("decode", "lazy"):
        Bn = case["B"]
        s["cache"] = _running_cache(case, g, cfg)
        s["cnn"] = _cnn(case, g, cfg)
        # the tokens that come in: one period of them, or sixteen in turn
        steps = case["window"] - 2 * _rho(case) if case["kind"] == "lazy" else 16
        s["q"], s["k"], s["v"] = (_normal(g, steps, Bn, h, case["D"], dtype=dt) for h in (case["Hq"], case["Hkv"], case["Hkv"]))
        s["steps"], s["at"] = steps, 0
        s["out"] = torch.zeros((steps if case["kind"] == "lazy" else 1, Bn, case["Hq"], case["D"]), dtype=dt, device="cuda")
        if case["kind"] == "lazy":
            s["ws"] = B.decode_workspace(cfg, None, Bn)
            s["ws_score"] = _bytes(B.ltea_rescore_workspace_bytes(cfg, s["cnn"], Bn))
        elif case["rope"]:
            s["k_feat"] = _normal(g, steps, Bn, case["Hkv"], case["D"], dtype=dt)
            freq = 10000.0 ** (-torch.arange(0, case["D"], 2, device="cuda", dtype=torch.float64) / case["D"])
            angle = torch.arange(131072, device="cuda", dtype=torch.float64)[:, None] * freq
            s["rope"] = B.upload_rope(angle.cos(), angle.sin())
            s["ws"] = _bytes(B.lib().ltea_decode_feat_workspace_bytes(ctypes.byref(cfg), ctypes.byref(s["cnn"].struct), Bn))
        elif not case["static"]:
            s["ws"] = B.decode_workspace(cfg, s["cnn"], Bn)
        return s
    lens = _lengths(case)
    total, longest = sum(lens), max(lens)
    s["q"], s["k"], s["v"] = _qkv(case, g, total)
    s["cu"], s["longest"] = _cu(lens), longest
    if case["kind"] == "append":
        old = [case["hist"]] * case["B"]
        q, k, v = _qkv(case, g, sum(old))
        cu = _cu(old)
        s["cnn"] = _cnn(case, g, cfg, k, v, cu, case["hist"])
        s["cache"] = B.alloc_cache(cfg, case["B"])
        B.ltea_prefill(cfg, s["cnn"], q, k, v, cu, case["hist"], s["cache"])
        s["ws"] = _bytes(B.ltea_append_workspace_bytes(cfg, s["cnn"], case["B"], total, longest))
        s["out"] = torch.zeros((total, case["Hq"], case["D"]), dtype=dt, device="cuda")
        return s
    # a rotary model scores its keys as they are before the rotation
    s["k_feat"] = _normal(g, total, case["Hkv"], case["D"], dtype=dt) if case.get("rope") else None
    s["cnn"] = _cnn(case, g, cfg, s["k"] if s["k_feat"] is None else s["k_feat"], s["v"], s["cu"], longest)
    if case["kind"] == "train":
        s["dout"] = _normal(g, total, case["Hq"], case["D"], dtype=dt)
        s["lam"] = torch.full((case["Hkv"],), 1e-3, device="cuda")
        s["ws"] = _bytes(B.ltea_train_workspace_bytes(cfg, s["cnn"], case["B"], total, longest))
        s["ws_cnn"] = _bytes(B.lib().ltea_cnn_backward_workspace_bytes(ctypes.byref(cfg), ctypes.byref(s["cnn"].struct), total))
        return s
    s["cache"] = B.alloc_cache(cfg, case["B"])
    s["ws"] = _bytes(B.ltea_workspace_bytes(cfg, s["cnn"], case["B"], total, longest))
    s["out"] = torch.zeros((total, case["Hq"], case["D"]), dtype=dt, device="cuda")
    return s


def run(s):
    cfg, kind = s["cfg"], s["kind"]
    if kind == "prefill":
        out = B.ltea_prefill(cfg, s["cnn"], s["q"], s["k"], s["v"], s["cu"], s["longest"], s["cache"], out=s["out"],
                             workspace=s["ws"], k_feat=s["k_feat"])
        return [out] + _cache_tensors(s["cache"])
    if kind == "append":
        out = B.ltea_prefill_append(cfg, s["cnn"], s["q"], s["k"], s["v"], s["cu"], s["longest"], s["cache"], out=s["out"],
                                    workspace=s["ws"])
        return [out] + _cache_tensors(s["cache"])
    if kind == "lazy":
        for i in range(s["steps"]):
            B.ltea_decode_step_lazy(cfg, s["q"][i], s["k"][i], s["v"][i], s["cache"], out=s["out"][i], workspace=s["ws"])
        B.ltea_rescore(cfg, s["cnn"], s["cache"], workspace=s["ws_score"])
        return [s["out"]] + _cache_tensors(s["cache"])
    if kind == "decode":
        i = s["at"]
        s["at"] = (i + 1) % s["steps"]
        q, k, v, out = s["q"][i], s["k"][i], s["v"][i], s["out"][0]
        if s["case"]["static"]:
            B.ltea_decode_step_static(cfg, s["cnn"], q, k, v, s["cache"], out)
        elif s["case"]["rope"]:
            B.ltea_decode_step_feat(cfg, s["cnn"], q, k, v, s["cache"], rope=s["rope"], k_feat=s["k_feat"][i], out=out,
                                    workspace=s["ws"])
        else:
            B.ltea_decode_step(cfg, s["cnn"], q, k, v, s["cache"], out=out, workspace=s["ws"])
        return [out] + _cache_tensors(s["cache"])
    out, lse, logits, ws = B.ltea_train_forward(cfg, s["cnn"], s["q"], s["k"], s["v"], s["cu"], s["longest"], workspace=s["ws"])
    dq, dk, dv, dz, counts = B.ltea_train_backward(cfg, s["q"], s["k"], s["v"], s["cu"], s["longest"], out, s["dout"], lse,
                                                   logits, s["lam"], ws)
    dw, dbias, dw_out, db_out, dk_feat, dv_feat = B.ltea_cnn_backward(cfg, s["cnn"], s["k"], s["v"], s["cu"], s["longest"], dz,
                                                                 workspace=s["ws_cnn"])
    return [out, lse, logits, dq, dk, dv, dz, counts, dw, dbias, dw_out, db_out, dk_feat, dv_feat]
