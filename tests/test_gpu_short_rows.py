"""Short rows of calls run from the item table, several to a workgroup:
selections and traces against the oracle at the edges of the waves a row takes
(2048, 4096 and 8192 elements), of K, and of the kept entries' limit."""
import numpy as np
import pytest

from paper_2609_08450_amd import workloads as W
from tests.test_gpu_parity import parity, say, topk  # noqa: F401
from tests.test_gpu_teams import _pack

pytestmark = pytest.mark.gpu


def _row(rng, L, K, kind):
    x = rng.standard_normal(L)
    if kind == 1:                        # every value the same
        x[:] = -1.25
    elif kind == 2:                      # masked entries at the boundary
        x[rng.random(L) < 0.6] = -np.inf
    elif kind == 3:                      # few values, both zeros among them
        x = rng.choice(np.array([-1.0, -0.0, 0.0, 0.5, np.inf, -np.inf]), L)
    elif kind == 4:                      # distinct keys of one coarse bin
        x = rng.uniform(100.0, 100.4, L)
    elif kind == 5 and L > K + 70:       # 64 or 65 entries in the boundary bin
        pos = rng.permutation(L)
        n = 64 + L % 2
        x = rng.uniform(-2.0, -1.0, L)
        x[pos[:K - 1]] = rng.uniform(4.0, 9.0, K - 1)
        x[pos[K - 1:K - 1 + n]] = rng.uniform(2.001, 2.060, n)
    elif kind == 6:                      # past FP16's range, subnormals
        x *= rng.choice(np.array([1e-42, 1e-6, 1.0, 1e6, 3e38]), L)
        x = np.clip(x, -3.4e38, 3.4e38)
    return x.astype(np.float32)


@pytest.mark.parametrize("K", [1, 63, 300, 2048, 4096, 8000])
def test_rows_at_the_edges(topk, K):  # noqa: F811
    rng = np.random.default_rng(81 + K)
    edges = [0, 1, 2, 3, 5, 255, 256, 257, 2044, 2047, 2048, 2049, 4093, 4095, 4096, 4097, 6000,
             8188, 8191, 8192, 8193, 9000]
    edges += [max(0, K + d) for d in (-1, 0, 1, 2, 64)]
    rows = [_row(rng, L, K, kind) for kind in range(7) for L in edges]
    rows += [_row(rng, int(L), K, i % 7) for i, L in enumerate(rng.integers(0, 8192, 560))]
    order = rng.permutation(len(rows))
    rows = [rows[i] for i in order]
    _, st = parity(topk, _pack(rows, K, "short rows"), per_k=True, where=f"short rows K {K}")
    say(st)
    assert st["direct"] > 0 and st["exact_unsampled"] > 0


@pytest.mark.parametrize("case", ["low floor", "long rows", "index order"])
def test_where_short_rows_stay_alone(topk, case):  # noqa: F811
    """A sampling floor inside the short lengths, more long items than resident
    workgroups, and more rows than the table holds."""
    rng = np.random.default_rng(87)
    K, pol, n = 256, topk.default_policy(), 700
    lens = rng.integers(1, 8000, n)
    if case == "low floor":
        pol.l_samp_min = 3000
    elif case == "long rows":
        lens[:600] = rng.integers(8192, 12000, 600)
    else:
        lens = rng.integers(1, 600, 16400)
    rows = [_row(rng, int(L), K, i % 7) for i, L in enumerate(lens)]
    _, st = parity(topk, _pack(rows, K, case), policy=pol, where=case)
    say(st)
    assert st["exact_unsampled"] > 0
