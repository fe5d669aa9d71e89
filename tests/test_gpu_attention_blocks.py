"""Block schedule of the bf16 prefill attention: window lower edges and diagonals at every offset from the 32-key blocks,
compact segments whose positions are in no order, that end inside a block, that nobody or only some rows see, and that are
longer than the positions kept in LDS.  Against the fp64 oracle, at the output tolerance of the other attention tests."""
import numpy as np
import pytest
import torch

from oracle import ltea_oracle as orc
from paper_2510_20787_amd import binding as B
from paper_2510_20787_amd import workloads as wl
from .gpu_util import DeviceWorkload, dev, to_np, OUT_TOL

pytestmark = pytest.mark.gpu


# what a prefill leaves, what decode steps leave, and two orders in which the last blocks hold late positions or none but them
ORDERS = {"ascending": lambda p, rng: np.sort(p), "shuffled": lambda p, rng: rng.permutation(p),
          "descending": lambda p, rng: np.sort(p)[::-1].copy(),
          "runs": lambda p, rng: np.concatenate([np.sort(p)[r::3] for r in range(3)]), "as given": lambda p, rng: p}


def run(D, G, window, budget, lens, keep_of, order, seed):
    rng = np.random.default_rng(seed)
    w = wl.make_prefill("blocks", seed, "bf16", lens, 2 * G, 2, D, window, budget, qkv_scale=1.0)
    d = DeviceWorkload(w)
    cache = d.new_cache()
    for t in (cache.k_ret, cache.v_ret):
        t.fill_(float("nan"))                   # slots past the last entry are never used
    kq, vq = to_np(d.k), to_np(d.v)
    keep = {}
    for s, n in enumerate(lens):
        lo = int(w.cu_seqlens[s])
        for h in range(w.Hkv):
            p = np.asarray(keep_of(n, h, rng), np.int64)[:budget]
            keep[s, h] = np.sort(p)
            p = ORDERS[order](p, rng)
            m = len(p)
            cache.ret_count[s, h] = m
            cache.ret_pos[s, h, :m] = torch.from_numpy(p.astype(np.int32))
            cache.k_ret[s, h, :m] = dev(kq[lo + p, h], "bf16")
            cache.v_ret[s, h, :m] = dev(vq[lo + p, h], "bf16")
    out = to_np(B.ltea_sparse_attention(d.cfg, d.q, d.k, d.v, d.cu, d.max_seqlen, cache))
    cfg = orc.OracleCfg(w.Hq, w.Hkv, w.D, window, budget, 0, 0.0)
    for s, n in enumerate(lens):
        lo = int(w.cu_seqlens[s])
        ref = orc.sparse_attention_sequence(w.q[lo:lo + n], w.k[lo:lo + n], w.v[lo:lo + n], cfg, [keep[s, h] for h in range(w.Hkv)])
        err = np.abs(out[lo:lo + n] - ref).max()
        assert err <= OUT_TOL["bf16"] * min(1.0, np.abs(ref).max()), f"sequence {s}: {err}"


@pytest.mark.parametrize("D,G", [(64, 1), (64, 4), (128, 1), (128, 4)])
@pytest.mark.parametrize("window", [1, 17, 31, 32, 33, 63, 64, 65, 96, 127, 200])
def test_window_edges(D, G, window):
    """Sequences that end at, before and after block and tile ends; two compact blocks, the second one cut short."""
    run(D, G, window, 40, [1, 31, 33, 129, 290], lambda n, h, rng: np.arange(h, n, 5 + h), "ascending", window)


@pytest.mark.parametrize("D,G", [(64, 1), (64, 4), (128, 1)])
@pytest.mark.parametrize("budget", [1, 31, 32, 33, 95, 128, 300])
@pytest.mark.parametrize("order", ["ascending", "shuffled", "descending", "runs"])
def test_compact_segments(D, G, budget, order):
    """Odd and even numbers of window and compact blocks, blocks that nobody or only some rows see; one head that keeps nothing."""
    run(D, G, 64, budget, [420, 97, 230], lambda n, h, rng: [] if h == 1 and n == 230 else rng.permutation(n)[:2 * n // 3], order, budget)


@pytest.mark.parametrize("D,G", [(64, 1), (128, 4)])
@pytest.mark.parametrize("order", ["ascending", "shuffled", "runs"])
def test_segments_longer_than_lds(D, G, order):
    """More than 2048 and more than 4096 entries: several groups of 64 blocks."""
    run(D, G, 33, 4500, [4700], lambda n, h, rng: np.sort(rng.permutation(n)[:4400 - 2100 * h]), order, 3)


@pytest.mark.parametrize("D,G", [(64, 1), (64, 4), (128, 1), (128, 4)])
@pytest.mark.parametrize("n,window,runs", [(277, 96, 3), (330, 97, 2), (421, 64, 4), (161, 128, 3)])
def test_late_entries_in_interleaved_runs(D, G, n, window, runs):
    """The segment's last blocks hold only positions behind the window of rows past the sequence's end: no wave may take them
    (the others would not load and wait for those tiles)."""
    late = np.arange(n - window, n)
    order = np.concatenate([late[r::runs] for r in range(runs)])
    run(D, G, window, window, [n, n - 32], lambda m, h, rng: order[order < m], "as given", runs)


@pytest.mark.parametrize("D,G", [(64, 1), (64, 4), (128, 1)])
@pytest.mark.parametrize("entries", [2015, 2016, 2017, 2048, 2049, 4064, 4097])
def test_groups_of_64_blocks(D, G, entries):
    """Segments around the end of a group of 64 blocks (63 where the window takes an odd number), ascending and with the
    earliest positions in the last group, so that a group that nobody sees comes before one that all rows see."""
    late_first = lambda n: np.concatenate([np.arange(n // 2, n), np.arange(n // 2)])[-entries:]
    run(D, G, 40 + entries % 64, entries, [4200], lambda n, h, rng: np.arange(entries) if h == 0 else late_first(n), "as given", 5)
