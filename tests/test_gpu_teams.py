"""Rows whose exact route is run by a team of workgroups: calls without a
sampled row (K from 4352 up) cut into segments, and split rows whose sampled
proposal fails.  Selections and traces against the oracle; with one poll per
bounded wait the teams break up and the last member runs the row alone."""
import numpy as np
import pytest

from paper_2609_08450_amd import workloads as W
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


@pytest.mark.parametrize("n", [33, 80, 150, 300])
def test_every_member_is_resident(topk, n):  # noqa: F811
    """Row counts between the powers of two, the long rows all on one die (every
    eighth): no member waits in vain."""
    rng = np.random.default_rng(79 + n)
    K = 4400
    lens = np.where(np.arange(n) % 8 == 0, rng.integers(60000, 131072, n),
                    rng.integers(4401, 12000, n))
    wl = _pack([W.decode_mixture_row(rng, int(L)) for L in lens], K, "one die")
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
