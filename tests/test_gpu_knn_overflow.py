"""Matrix-core kNN over a base whose sampled rows are all far: nearly every later row passes the
first threshold, the buffers overflow, and the scan answers.  Bases of one stage beside it."""
import math

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def B():
    from paper_2201_13007_amd import binding
    binding.lib()
    return binding


def compare(B, base, q, k, label):
    print(f"case: {label} n={base.shape[0]} nq={len(q)} k={k}", flush=True)
    ids, d, path = B.knn(torch.from_numpy(base).cuda(), torch.from_numpy(q).cuda(), k, return_path=True)
    eids, ed = oracle.knn(base, q, k)
    np.testing.assert_array_equal(ids.cpu().numpy(), eids)
    np.testing.assert_array_equal(d.cpu().numpy(), ed)
    assert path == "mfma"


@pytest.mark.parametrize("nq", [5, 300])
@pytest.mark.parametrize("integer", [True, False])
def test_far_sample(B, nq, integer):
    rng = np.random.default_rng(nq)
    n, d = 20_000, 32
    base = rng.integers(0, 10, (n, d)).astype(np.float32)
    q = rng.integers(0, 10, (nq, d)).astype(np.float32)
    # the rows of the first 16 tiles: offset o of tile t holds row o ntile + (t mul) mod ntile
    ntile = (n + 127) // 128 * 2
    mul = max(1, int(0.6180339887498949 * ntile))
    while math.gcd(mul, ntile) != 1:
        mul += 1
    rows = (np.arange(64)[:, None] * ntile + (np.arange(16) * mul % ntile)[None, :]).ravel()
    rows = rows[rows < n]
    base[rows] += 200
    q[::2] += 1      # (some of the queries among the others, some nearer to none)
    if not integer:
        base += rng.random((n, d)).astype(np.float32) / 4
    compare(B, base, q, 10, "far sample")


# one stage: up to 2,048 rows and 255 queries; lists of up to 64 by a wavefront
@pytest.mark.parametrize("n", [1023, 1025, 2048, 2049])
@pytest.mark.parametrize("nq", [1, 255, 256])
@pytest.mark.parametrize("k", [1, 64, 65, 96])
def test_one_stage(B, n, nq, k):
    rng = np.random.default_rng([n, nq, k])
    base = rng.integers(0, 30, (n, 36)).astype(np.float32)
    compare(B, base, rng.integers(0, 30, (nq, 36)).astype(np.float32), k, "one stage")
