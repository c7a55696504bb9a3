"""The forms of the general kernel by launch size: few queries (all resident with the most
registers), some, and many, at the smallest and largest list of each number of slots."""
import numpy as np
import pytest

from test_gpu_search_forms import check, graph

pytestmark = pytest.mark.gpu
pytest.importorskip("torch")


@pytest.mark.parametrize("copies", [1, 200, 1200])      # of 6 queries
@pytest.mark.parametrize("M,L", [(1, 64), (2, 1), (2, 64), (2, 65), (2, 128), (2, 129), (2, 256), (2, 257), (2, 384), (2, 385),
                                 (2, 512), (2, 513), (3, 40), (3, 200), (4, 1), (4, 100), (4, 300), (4, 600), (5, 60),
                                 (5, 120), (6, 130), (7, 400), (8, 64), (12, 100)])
def test_general_kernel(M, L, copies):
    g = np.random.default_rng([L, M])
    n = 6000
    base = g.integers(0, 16, (n, 16)).astype(np.float32)
    q = g.integers(0, 16, (6, 16)).astype(np.float32)
    check(base, graph(n, 40, g), q, min(L, 20), L, M, "adaptive", repeat=copies, label="launch size",
          ws_hash_slots=1 << 14 if copies > 200 else 1 << 16, lds_hash_slots=4096 if M != 2 else 0,
          orc={"rho": 0.7, "staged": bool(L % 2)})


@pytest.mark.parametrize("copies", [1, 200, 900])
@pytest.mark.parametrize("d,dtype", [(260, "f32"), (960, "f32"), (960, "bf16"), (200, "fp8")])
def test_general_kernel_rows(d, dtype, copies):
    g = np.random.default_rng(d)
    base = g.standard_normal((900, d)).astype(np.float32)
    q = g.standard_normal((6, d)).astype(np.float32)
    for M, L in ((2, 50), (2, 300), (4, 100), (6, 70)):
        check(base, graph(900, 32, g), q, 10, L, M, "static", "l2", dtype, exact=False, repeat=copies,
              label="launch size, rows", orc={"static_I": 2})
