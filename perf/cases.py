"""The calls whose time is measured: ragged exact Top-K as a serving program makes it.

A case is one call (or one captured step of several calls) of the public entry
points in ``paper_2609_08450_amd.topk`` on score rows already on the GPU.  The
fields of a case:

  rows, lo, hi   row count and the range of the row lengths
  spread         how the lengths lie in it: "uniform", "log" (log-uniform),
                 or "causal" (row i of a prefill block: hi - rows + 1 + i, in
                 a buffer of pitch hi)
  K              selected entries per row
  scores         "normal", "mixture" (decode rows), "indexer" (a prefill
                 block's products), "ties" (a codebook), "edge" (edge mix)
  calls          1: an eager call through a TopK holder that the program
                 keeps; more: that many layers' calls of the allocation-free
                 entry point, captured in one graph that is replayed

Row lengths follow from the case alone; the scores follow from the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2609_08450_amd import topk

VIEW_STRIDE = 128  # stride of the strided rows of the edge mix


def listed():
    return [
        # a debug prompt or a small model: latency and launches are all of it
        dict(name="tiny", rows=4, lo=1024, hi=8192, spread="uniform", K=256,
             scores="normal", calls=1),
        # one user at a long context: one row over the whole chip
        dict(name="decode_one", rows=1, lo=131071, hi=131071, spread="uniform", K=2048,
             scores="mixture", calls=1),
        # the decode batch of the benchmark
        dict(name="decode", rows=64, lo=16384, hi=131072, spread="uniform", K=2048,
             scores="mixture", calls=1),
        # a decode step as serving runs it: several layers in one graph
        dict(name="decode_step", rows=32, lo=4096, hi=65536, spread="uniform", K=1024,
             scores="mixture", calls=8),
        # a large decode batch of short selections
        dict(name="decode_wide", rows=256, lo=8192, hi=131072, spread="uniform", K=512,
             scores="mixture", calls=1),
        # the decode batch with wider selections: the largest K that is
        # sampled, and one that takes the exact route
        dict(name="decode_k4096", rows=64, lo=16384, hi=131072, spread="uniform", K=4096,
             scores="mixture", calls=1),
        dict(name="decode_k8192", rows=64, lo=16384, hi=131072, spread="uniform", K=8192,
             scores="mixture", calls=1),
        # scores of few distinct values: ties at the boundary in every row
        dict(name="decode_ties", rows=64, lo=16384, hi=131072, spread="uniform", K=2048,
             scores="ties", calls=1),
        # the first chunk of a prefill: every length from 1 up
        dict(name="prefill_first", rows=4096, lo=1, hi=4096, spread="causal", K=2048,
             scores="indexer", calls=1),
        # the last chunk of a long prefill: the largest call
        dict(name="prefill", rows=4096, lo=126977, hi=131072, spread="causal", K=2048,
             scores="indexer", calls=1),
        # mixed traffic: direct rows, ties, strided rows, masked entries
        dict(name="edge_mix", rows=1024, lo=512, hi=262144, spread="log", K=2048,
             scores="edge", calls=1),
        # few rows at contexts of up to a million tokens
        dict(name="long_split", rows=16, lo=524288, hi=1048576, spread="uniform", K=2048,
             scores="mixture", calls=1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges, at most about a quarter of the
    largest listed one's scores."""
    kind = rng.choice(["decode", "decode", "step", "long", "prefill", "first", "edge", "ties"])
    K = rng.choice([_log_int(rng, 64, 16384), _log_int(rng, 256, 4096), 2048])
    if kind == "decode":
        hi = _log_int(rng, 2048, 262144)
        rows = min(_log_int(rng, 1, 512), max(1, (1 << 25) // hi))
        return dict(rows=rows, lo=max(1, int(hi * rng.uniform(0.05, 1.0))), hi=hi,
                    spread="uniform", K=K, scores=rng.choice(["mixture", "mixture", "normal"]),
                    calls=1)
    if kind == "step":
        hi = _log_int(rng, 4096, 131072)
        return dict(rows=_log_int(rng, 1, 64), lo=hi // rng.randint(2, 9), hi=hi, spread="uniform",
                    K=min(K, 4096), scores="mixture", calls=rng.randint(2, 6))
    if kind == "long":
        hi = _log_int(rng, 262144, 1048576)
        return dict(rows=rng.randint(1, 24), lo=int(hi * rng.uniform(0.3, 1.0)), hi=hi,
                    spread="uniform", K=K, scores="mixture", calls=1)
    if kind == "prefill":
        hi = _log_int(rng, 8192, 131072)
        rows = min(_log_int(rng, 513, 8192), hi, (1 << 27) // hi)
        return dict(rows=rows, lo=hi - rows + 1, hi=hi, spread="causal", K=min(K, 8192),
                    scores="indexer", calls=1)
    if kind == "first":
        rows = _log_int(rng, 513, 8192)
        return dict(rows=rows, lo=1, hi=rows, spread="causal", K=min(K, 4096), scores="indexer",
                    calls=1)
    if kind == "edge":
        return dict(rows=_log_int(rng, 64, 1024), lo=rng.randint(300, 900),
                    hi=_log_int(rng, 16384, 262144), spread="log", K=min(K, 4096), scores="edge",
                    calls=1)
    hi = _log_int(rng, 8192, 131072)
    return dict(rows=_log_int(rng, 1, 128), lo=int(hi * rng.uniform(0.1, 1.0)), hi=hi,
                spread="uniform", K=min(K, 8192), scores="ties", calls=1)


def _lengths(case):
    n, lo, hi = case["rows"], case["lo"], case["hi"]
    if case["spread"] == "causal":
        return (hi - n + 1 + np.arange(n)).astype(np.int32)
    g = np.random.default_rng([n, lo, hi])
    if case["spread"] == "log":
        x = np.exp(g.uniform(math.log(lo), math.log(hi), n))
        if case["scores"] == "edge":  # every fourth row is no longer than K
            short = np.exp(g.uniform(math.log(min(lo, case["K"])), math.log(case["K"]), n))
            x = np.where(np.arange(n) % 4 == 0, np.floor(short), x)
        return np.clip(x, 1, hi).astype(np.int32)
    return g.integers(lo, hi, size=n, endpoint=True).astype(np.int32)


def _offsets(case, lens):
    if case["spread"] == "causal":
        return np.arange(len(lens), dtype=np.int64) * case["hi"]
    return np.concatenate([[0], np.cumsum(lens[:-1], dtype=np.int64)]).astype(np.int64)


def _positions(lens, offs):
    """Row and row-relative index of every element of a packed buffer."""
    n = torch.from_numpy(lens).cuda().long()
    row = torch.repeat_interleave(torch.arange(len(lens), device="cuda"), n)
    return row, torch.arange(row.numel(), device="cuda") - torch.from_numpy(offs).cuda()[row]


def _randn(n, g):
    return torch.randn(n, generator=g, device="cuda")


def _mixture(lens, offs, g):
    """N(0,1), a recency term toward the row end, and one block of 64
    positions in a hundred around 3."""
    total = int(lens.sum())
    row, i = _positions(lens, offs)
    last = torch.from_numpy(lens - 1).cuda()[row]
    x = _randn(total, g) + 0.5 * torch.exp((i - last).float() / 4096.0)
    hot = torch.rand(total // 64 + 1, generator=g, device="cuda") < 0.01
    return torch.where(hot.repeat_interleave(64)[:total], 3.0 + 0.5 * _randn(total, g), x)


def _books(n, g):
    """n codebooks of 256 values: the lowest of 4096 N(0,1) draws, so that
    about a dozen of them share the leading bits of a 16-bit float."""
    return torch.randn((n, 4096), generator=g, device="cuda").sort(dim=1).values[:, :256]


def _ties(lens, offs, g):
    row, _ = _positions(lens, offs)
    pick = torch.randint(0, 256, (row.numel(),), generator=g, device="cuda")
    return _books(len(lens), g)[row, pick].contiguous()


def _edge(lens, offs, g):
    """By row mod 4: N(0,1) no longer than K; 256 distinct values; lower
    values on one residue of every 128 positions; -inf with probability 0.3."""
    total = int(lens.sum())
    row, i = _positions(lens, offs)
    x = _randn(total, g)
    books = torch.randn((len(lens), 256), generator=g, device="cuda")
    pick = torch.randint(0, 256, (total,), generator=g, device="cuda")
    x = torch.where(row % 4 == 1, books[row, pick], x)
    phase = [int(format(r % VIEW_STRIDE, "07b")[::-1], 2) for r in range(len(lens))]
    on = i % VIEW_STRIDE == torch.tensor(phase, device="cuda")[row]
    x = torch.where((row % 4 == 2) & on, x - 2.0, x)
    masked = (row % 4 == 3) & (torch.rand(total, generator=g, device="cuda") < 0.3)
    return torch.where(masked, torch.full_like(x, -math.inf), x)


def _indexer(rows, context, g, dim=64, heads=8):
    """sum_h w_h relu(q_h . k_j / sqrt(dim)), keys and weights shared."""
    keys = torch.randn((dim, context), generator=g, device="cuda")
    q = torch.randn((heads, rows, dim), generator=g, device="cuda")
    w = torch.rand(heads, generator=g, device="cuda").tolist()
    out = torch.zeros((rows, context), device="cuda")
    for r in range(0, rows, 512):
        for h in range(heads):
            d = torch.mm(q[h, r:r + 512], keys)
            out[r:r + 512] += d.clamp_(min=0).mul_(w[h] / math.sqrt(dim))
    return out.reshape(-1)


def _scores(case, lens, offs, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    if case["scores"] == "indexer":
        return _indexer(case["rows"], case["hi"], g)
    if case["scores"] == "normal":
        return _randn(int(lens.sum()), g)
    return {"mixture": _mixture, "ties": _ties, "edge": _edge}[case["scores"]](lens, offs, g)


class Selection(dict):
    """The outputs of a pass.  A call returns each row's K pairs in no
    particular order, and another order from one call to the next, so whoever
    reads them here gets them by index.  The pass itself has written both
    buffers: ordering them is no part of it."""

    def __getitem__(self, name):
        idx, order = torch.sort(dict.__getitem__(self, "idx"), dim=-1, stable=True)
        return idx if name == "idx" else torch.gather(dict.__getitem__(self, "val"), -1, order)


def prepare(case, seed):
    lens = _lengths(case)
    offs = _offsets(case, lens)
    n, K, calls = case["rows"], case["K"], case["calls"]
    layers = [_scores(case, lens, offs, seed * 64 + layer) for layer in range(calls)]
    state = {
        "layers": layers,
        "offs": torch.from_numpy(offs).cuda(),
        "lens": torch.from_numpy(lens).cuda(),
        "idx": torch.empty((calls * n, K), dtype=torch.int32, device="cuda"),
        "val": torch.empty((calls * n, K), dtype=torch.float32, device="cuda"),
    }
    if calls == 1:
        state["topk"] = topk.TopK(n, K)
        return state

    def step():
        for layer, x in enumerate(layers):
            topk.topk_ragged_noalloc(x, state["offs"], state["lens"], n, K,
                                     state["idx"][layer * n:(layer + 1) * n],
                                     state["val"][layer * n:(layer + 1) * n])

    step()  # the library's own workspace is set up outside the capture
    torch.cuda.synchronize()
    state["graph"] = torch.cuda.CUDAGraph()
    with torch.cuda.graph(state["graph"]):
        step()
    return state


def run(state):
    if "graph" in state:
        state["graph"].replay()
    else:
        state["topk"](state["layers"][0], state["offs"], state["lens"], state["idx"], state["val"])
    return Selection(idx=state["idx"], val=state["val"])


def work(case):
    """Every valid score read once, every output written once, and the row
    table; the selection's compares are not counted as operations."""
    lens = _lengths(case).astype(np.int64)
    n, K = case["rows"], case["K"]
    return {"bytes": case["calls"] * (4 * int(lens.sum()) + 8 * K * n + 12 * n), "flops": 0}


def tolerance(case):
    """The selection is defined to the last bit: values are copies of the
    scores, and ties go to the lowest index."""
    return "exact"


def exact(case, seed):
    """The selection by its definition: the K largest of the keys (value,
    then lowest index), by index."""
    lens = _lengths(case)
    offs = _offsets(case, lens)
    n, K, calls = case["rows"], case["K"], case["calls"]
    idx = torch.full((calls * n, K), -1, dtype=torch.int64, device="cuda")
    val = torch.full((calls * n, K), -math.inf, dtype=torch.float64, device="cuda")
    for layer in range(calls):
        x = _scores(case, lens, offs, seed * 64 + layer)
        for r in range(n):
            s = x[int(offs[r]):int(offs[r]) + int(lens[r])]
            L = s.numel()
            if L <= K:
                i = torch.arange(L, device="cuda")
            else:
                b = s.view(torch.int32).long()
                key = torch.where(b < 0, -(b & 0x7FFFFFFF) - 1, b)  # -0.0 below +0.0
                key = (key << 31) + (0x7FFFFFFF - torch.arange(L, device="cuda"))
                i = torch.topk(key, K, sorted=False).indices.sort().values
            k = layer * n + r
            idx[k, K - i.numel():] = i
            val[k, K - i.numel():] = s[i].double()
    return {"idx": idx, "val": val}
