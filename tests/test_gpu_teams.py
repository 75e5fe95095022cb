"""Rows whose exact route is run by a team of workgroups: calls without a
sampled row (K from 4352 up) cut into segments, and split rows whose sampled
proposal fails.  Selections and traces against the oracle; with one poll per
bounded wait the teams break up and the last member runs the row alone."""
import numpy as np
import pytest

import oracle
from paper_2609_08450_amd import workloads as W
from tests.gpu_util import assert_same_selection, device_arrays
from tests.test_gpu_parity import _reread_rows, parity, say, topk  # noqa: F401

pytestmark = pytest.mark.gpu


def _pack(rows, K, name):
    rows = [np.asarray(x, np.float32) for x in rows]
    lens = np.array([x.size for x in rows], np.int32)
    gap = np.arange(len(rows)) % 4            # every 4-byte alignment
    offs = (np.cumsum(lens + gap) - lens).astype(np.int64)
    buf = np.zeros(int(offs[-1] + lens[-1]), np.float32)
    for o, x in zip(offs, rows):
        buf[o:o + x.size] = x
    return W.Workload(name, buf, offs, lens, K, "")


def _rows(rng, L, K, kind):
    if kind == "mixture":
        return W.decode_mixture_row(rng, L)
    if kind == "equal":                       # key windows, then index windows
        return np.full(L, 0.5)
    if kind == "masked":                      # fewer finite values than K
        x = np.full(L, -np.inf)
        x[rng.choice(L, K // 2, replace=False)] = rng.standard_normal(K // 2)
        return x
    if kind == "one bin":                     # distinct keys of one coarse bin
        return rng.uniform(100.0, 100.9, L)
    if kind == "codes":                       # 64 values, some of one bin
        return rng.choice(np.linspace(1.0, 1.2, 64), L)
    # a boundary bin of exactly n entries, K ending inside it
    n = int(kind)
    x = rng.uniform(-2.0, -1.0, L)
    pos = rng.choice(L, K - 7 + n, replace=False)
    x[pos[:K - 7]] = rng.uniform(4.0, 9.0, K - 7)
    x[pos[K - 7:]] = rng.uniform(2.001, 2.060, n)
    return x


@pytest.mark.parametrize("spin", [0, 1], ids=["waits", "one-poll"])
@pytest.mark.parametrize("K", [4352, 8192, 16384])
def test_calls_without_a_sampled_row(topk, K, spin):  # noqa: F811
    """Lengths around one workgroup's row, around whole chunks and segments,
    and streamed ranges; boundary bins at the kept sets' limits (1024 for one
    workgroup, 6144 for a team)."""
    rng = np.random.default_rng(71 + K)
    small = [K, K + 1, max(K + 1, 8192), max(K + 1, 16383), max(K + 1, 16385)]
    rows = [_rows(rng, L, K, k) for L in small for k in ("mixture", "equal")]
    for L in (24576, 32769, 65535, 131072, 200001):
        rows += [_rows(rng, L, K, k) for k in ("mixture", "equal", "masked", "one bin", "codes")]
    for L, kinds in ((32768, ("1024", "1025", "6144")), (90001, ("6144", "6145", "9000"))):
        rows += [_rows(rng, L, K, k) for k in kinds]
    topk.debug_set_spin_limit(spin)
    try:
        _, st = parity(topk, _pack(rows, K, "exact teams"), per_k=True, where=f"K {K} spin {spin}")
        # two rows: the whole chip for each, most members of a team
        _, st2 = parity(topk, _pack([_rows(rng, 700001, K, "mixture"), _rows(rng, 524288, K, "codes")],
                                    K, "large teams"), per_k=True, where=f"K {K} two rows")
    finally:
        topk.debug_set_spin_limit(0)
    say(st, st2)
    assert st["reread"] > 0
    assert (st["wait_fallback"] > 0) == bool(spin)


@pytest.mark.parametrize("spin", [0, 1], ids=["waits", "one-poll"])
@pytest.mark.parametrize("n", [5, 40])
def test_failed_proposals_of_split_rows(topk, n, spin):  # noqa: F811
    """Split rows of a call without an item table: underfilled, overflowing
    (with and without a boundary bin beyond the frontier), and rows around the
    verdict's thresholds, next to rows that certify."""
    rng = np.random.default_rng(73 + n)
    K = 2048
    rows = []
    for i in range(n):
        L = int(rng.integers(70000, 300000))
        x = W.decode_mixture_row(rng, L)
        phase = int(format(i % 128, "07b")[::-1], 2)
        on = x[phase::128].size
        kind = i % 6
        if kind == 0:                          # the view sees high values only: underfill
            x[phase::128] = rng.normal(4.0, 0.1, on)
        elif kind == 1:                        # and low ones only: overflow
            x[phase::128] = rng.normal(-2.0, 1.0, on)
        elif kind == 2:                        # ties past the frontier at the boundary
            x[rng.choice(L, 9000, replace=False)] = np.partition(x, L - K)[L - K] + np.float32(0.01)
        elif kind == 3:                        # the view a little high: around K admitted
            x[phase::128] += np.float32(0.25)
        elif kind == 4:                        # a little low: around the frontier
            x[phase::128] -= np.float32(0.35)
        rows.append(x)
    extra = _reread_rows(rng)
    rows += list(extra.values())
    topk.debug_set_spin_limit(spin)
    try:
        _, st = parity(topk, _pack(rows, K, "failed proposals"), where=f"{n} rows spin {spin}")
        _, st1 = parity(topk, _pack(rows, K, "failed proposals"), trace=False, where="again")
    finally:
        topk.debug_set_spin_limit(0)
    say(st)
    assert st["exact_underfill"] > 0 and st["exact_overflow"] > 0 and st["reread"] > 0
    if spin:
        assert st["wait_fallback"] > 0


def _skewed(seed, n, K=4400):
    rng = np.random.default_rng(seed)
    lens = np.where(np.arange(n) % 8 == 0, rng.integers(60000, 131072, n),
                    rng.integers(K + 1, 12000, n))
    return _pack([W.decode_mixture_row(rng, int(L)) for L in lens], K, "one die")


@pytest.mark.parametrize("n", [33, 80, 150, 170, 256])
def test_every_member_is_resident(topk, n):  # noqa: F811
    """Row counts up to the last that forms teams, the long rows all on one die
    (every eighth): no member waits in vain."""
    wl = _skewed(79 + n, n)
    for _ in range(3):
        _, st = parity(topk, wl, per_k=True, where=f"{n} rows")
        say(st)
        assert st["wait_fallback"] == 0


@pytest.mark.parametrize("n,every,long,short", [
    (12, 4, 500000, 4000), (24, 8, 262144, 4000), (48, 8, 262144, 30000),
    (96, 8, 131072, 4000), (300, 8, 65536, 9000), (400, 8, 131072, 4000)])
def test_segments_stay_for_running_ones_only(topk, n, every, long, short):  # noqa: F811
    """Tied sampled rows whose grid is larger than the resident workgroups, the
    long rows all on one or two dies: no staying segment waits in vain for one
    that needs its slot."""
    rng = np.random.default_rng(83 + n)
    rows = []
    for i in range(n):
        book = np.sort(rng.standard_normal(4096))[:256]
        rows.append(rng.choice(book, long if i % every == 0 else short))
    wl = _pack(rows, 2048, "one die, tied")
    for k in range(3):
        _, st = parity(topk, wl, trace=False, where=f"{n} rows")
        say(st)
        assert k == 0 or st["wait_fallback"] == 0


@pytest.mark.parametrize("n", [257, 300, 512])
def test_no_sampled_row_one_workgroup_each(topk, n):  # noqa: F811
    """Calls of more rows than CUs without a sampled row: a workgroup a row."""
    parity(topk, _skewed(89 + n, n), per_k=True, where=f"{n} rows")


def _team_calls(seed):
    """Calls whose rows are run by teams: without a sampled row, and tied ones
    (n, K as of the call)."""
    rng = np.random.default_rng(seed)
    kinds = ("mixture", "equal", "one bin", "codes", "masked")
    exact = _pack([_rows(rng, int(rng.integers(30000, 200000)), 8192, k) for k in kinds + kinds],
                  8192, "no sampled row")
    tied = []
    for _ in range(12):
        book = np.sort(rng.standard_normal(4096))[:256]
        tied.append(rng.choice(book, int(rng.integers(70000, 200000))))
    return exact, _pack(tied, 2048, "tied")


def _check(wl, gi, gv, where):
    oi, ov = oracle.topk_ragged(wl.scores, wl.row_offsets, wl.row_lengths, wl.K)
    assert_same_selection(gi.cpu().numpy(), gv.cpu().numpy(), oi, ov, where=where)


def _buffers(wl):
    import torch

    n = wl.n_rows
    return (*device_arrays(wl), n, wl.K, torch.full((n, wl.K), -7, dtype=torch.int32, device="cuda"),
            torch.full((n, wl.K), 7.0, device="cuda"))


def test_team_state_across_calls(topk):  # noqa: F811
    """One workspace for calls of both kinds in turn, with broken-up teams (one
    poll per wait) between: each call finds the row state it needs."""
    import torch

    ws = topk.alloc_workspace(16, 8192)
    calls = [(w, _buffers(w)) for s in (97, 101) for w in _team_calls(s)]
    try:
        for step, spin in enumerate([0, 0, 1, 0, 1, 1, 0]):
            topk.debug_set_spin_limit(spin)
            for w, b in calls:
                b[5].fill_(-7)
                topk.topk_ragged(*b, ws)
                torch.cuda.synchronize()
                _check(w, b[5], b[6], f"{w.name} step {step} spin {spin}")
    finally:
        topk.debug_set_spin_limit(0)
    say(topk.read_stats(ws))


@pytest.mark.parametrize("noalloc", [False, True], ids=["workspace", "noalloc"])
def test_team_graph_replays(topk, noalloc):  # noqa: F811
    """Both kinds captured in one graph, replayed with eager calls on the same
    workspace between the replays."""
    import torch

    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ws = topk.alloc_workspace(16, 8192, torch.device("cuda", 0), stream)
        calls = [(w, _buffers(w)) for w in _team_calls(103)]

    def call(b):
        if noalloc:
            topk.topk_ragged_noalloc(*b, stream=stream)
        else:
            topk.topk_ragged(*b, ws, stream)

    for _, b in calls:
        call(b)
    stream.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        for _, b in calls:
            call(b)
    for rep in range(3):
        with torch.cuda.stream(stream):
            for _, b in calls:
                b[5].fill_(-7)
            g.replay()
        stream.synchronize()
        for w, b in calls:
            _check(w, b[5], b[6], f"{w.name} replay {rep}")
            b[5].fill_(-7)
        torch.cuda.synchronize()
        for w, b in calls[::-1]:
            call(b)
        stream.synchronize()
        for w, b in calls:
            _check(w, b[5], b[6], f"{w.name} eager after replay {rep}")


def test_teams_on_two_streams(topk):  # noqa: F811
    """Two such calls at once, each with a stream and workspace of its own:
    members of one may keep the other's from running until a wait ends."""
    import torch

    streams = (torch.cuda.Stream(), torch.cuda.Stream())
    work = []
    for k, st in enumerate(streams):
        with torch.cuda.stream(st):
            ws = topk.alloc_workspace(16, 8192, torch.device("cuda", 0), st)
            work.append([(w, _buffers(w), ws, st) for w in _team_calls(107 + k)])
    torch.cuda.synchronize()
    for rep in range(4):
        for pair in zip(*work):
            for w, b, ws, st in pair:
                topk.topk_ragged(*b, ws, st)
    torch.cuda.synchronize()
    for one in work:
        for w, b, _, _ in one:
            _check(w, b[5], b[6], f"{w.name} on two streams")
