"""The staged matrix-core kNN at the edges of its tiles, stages and splits: every result must
be the oracle's (integer data) bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle
from paper_2201_13007_amd import synth


@pytest.fixture(scope="module")
def B():
    from paper_2201_13007_amd import binding
    binding.lib()
    return binding


def _check(B, base, q, k, metric="l2", self_join=False):
    qd = None if self_join else torch.from_numpy(q).cuda()
    ids, d, path = B.knn(torch.from_numpy(base).cuda(), qd, k, metric=metric, exclude_self=self_join, return_path=True)
    eids, ed = oracle.knn(base, base if self_join else q, k, metric=metric, exclude_self=self_join)
    np.testing.assert_array_equal(ids.cpu().numpy(), eids)
    np.testing.assert_array_equal(d.cpu().numpy(), ed)
    return path


# rows: less than a tile, tile and stage edges, several stages; queries: one, and the edges of
# the one-, two- and four-wavefront workgroups, and the plan for many queries (4096 up)
@pytest.mark.parametrize("n,nq", [(1, 1), (63, 3), (64, 64), (65, 65), (129, 128), (1024, 129), (1025, 256),
                                  (3000, 257), (20_011, 5), (2_500, 4_100)])
def test_knn_integer_tile_edges(B, n, nq):
    w = synth.integer_grid(n, 36, nq, lo=-9, hi=10, config=94)
    for k in (1, 24, 100):
        print(f"case: staged knn int n={n} nq={nq} k={k}", flush=True)
        assert _check(B, w.base, w.queries, k) == "mfma"


@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("lo,hi", [(0, 40), (200, 256)])
def test_knn_integer_folded_or_not(B, lo, hi, metric):
    # |x|^2 + 2 |q| |x| below 2^24 (small values) or above it (d = 256, values near 255)
    w = synth.integer_grid(4_000, 256, 40, lo=lo, hi=hi, config=95)
    print(f"case: staged knn int d=256 [{lo}, {hi}) {metric}", flush=True)
    assert _check(B, w.base, w.queries, 10, metric) == "mfma"


def test_knn_integer_ties_self_join(B):
    # few distinct distances: almost every product reaches the bound and ids decide
    w = synth.integer_grid(9_000, 4, 1, hi=3, config=96)
    print("case: staged knn int self-join, ties", flush=True)
    assert _check(B, w.base, None, 30, self_join=True) == "mfma"


def sample_rows(n):
    """Rows of the first stage of a call with few queries (knn_tile.h: position 64 t + o holds
    row o * ntile + (t * mul) % ntile)."""
    ntile = (n + 127) // 128 * 2
    mul = max(1, int(0.6180339887498949 * ntile))
    while np.gcd(mul, ntile) != 1:
        mul += 1
    off = (np.arange(min(ntile, 16)) * mul) % ntile
    rows = (np.arange(64)[:, None] * ntile + off[None, :]).ravel()
    return rows[rows < n]


def test_knn_integer_overflow_is_rescued(B):
    # the first stage's rows are all far away and the others all near: every later row beats
    # the bound, the buffers overflow, and the scan answers
    w = synth.integer_grid(9_000, 16, 7, hi=60, config=97)
    base = w.base.copy()
    base[sample_rows(9_000)] = 255.0
    print("case: staged knn int, overflowing buffers", flush=True)
    assert _check(B, base, w.queries, 50) == "mfma"


# float data: the resident kernels (d <= 128) and the wide one, each at its tile, stage and
# query-block edges; k = 100 and 256 take longer candidate lists (from 2048 rows up)
@pytest.mark.parametrize("d", [20, 64, 96, 128, 132, 384])
@pytest.mark.parametrize("n,nq", [(1, 2), (65, 64), (130, 129), (2048, 257), (3001, 70)])
def test_knn_float_tile_edges(B, d, n, nq):
    w = synth.deep_like(n=n, nq=nq, d=d, ncomp=8)
    for k, metric in ((1, "ip"), (10, "l2"), (96, "l2"), (100, "ip"), (256, "l2")):
        if k > 96 and n < 2048:
            continue
        print(f"case: staged knn float n={n} d={d} nq={nq} k={k} {metric}", flush=True)
        assert _check(B, w.base, w.queries, k, metric) == "mfma"


def test_knn_float_many_queries(B):
    # the plan for 4096 queries and more, and a self-join
    w = synth.tiny(n=5_000, nq=4_200, d=24)
    print("case: staged knn float 5000x24, 4200 queries", flush=True)
    assert _check(B, w.base, w.queries, 12) == "mfma"
    print("case: staged knn float 5000x24 self-join", flush=True)
    assert _check(B, w.base, None, 40, self_join=True) == "mfma"


@pytest.mark.parametrize("bad", [np.nan, np.inf, 1e-25])
def test_knn_float_values_for_the_scan(B, bad):
    # one value that the matrix cores cannot take sends the call to the scan
    w = synth.deep_like(n=2100, nq=20, d=96, ncomp=8)
    base = w.base.copy()
    base[1234, 7] = bad
    print(f"case: staged knn float with {bad}", flush=True)
    dev = torch.from_numpy(base).cuda(), torch.from_numpy(w.queries).cuda()
    ids, d, path = B.knn(*dev, 10, metric="ip", return_path=True)
    sids, sd = B.knn(*dev, 10, metric="ip", path="scan")
    assert path == "scan"
    assert torch.equal(ids, sids)
    np.testing.assert_array_equal(d.cpu().numpy(), sd.cpu().numpy())


def test_knn_float_overflow_is_rescued(B):
    w = synth.deep_like(n=9_000, nq=7, d=96, ncomp=8)
    base = w.base.copy()
    base[sample_rows(9_000)] += 100.0
    print("case: staged knn float, overflowing buffers", flush=True)
    assert _check(B, base, w.queries, 50) == "mfma"
    assert B.knn_last_rescanned() == 7
