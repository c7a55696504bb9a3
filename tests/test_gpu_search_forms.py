"""The forms of the one- and two-walker search against the oracle: few queries (up to eight
vectors per lane group in flight, all queue slots exchanged at once) and many, with the LDS
visited set roomy, overflowing into the workspace table, or absent, at the edges of the
vector layouts (1 to 64 lanes per vector, chunks past the row's end) and of the queue slots."""
import numpy as np
import pytest

import oracle
import parity

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
MANY = 8200    # more queries than can be resident at once in any form
FIELDS = ("global_steps", "substeps", "expansions", "dist_comps", "merges")


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def graph(n, R, g):
    """Random rows, each vertex linked to its neighbours on a ring too (all reachable)."""
    adj = g.integers(0, n, (n, R)).astype(np.int32)
    adj[:, 0] = (np.arange(n) + 1) % n
    adj[:, 1] = (np.arange(n) - 1) % n
    return adj


def check(base, adj, q, k, L, M, sync, metric="l2", dtype="f32", exact=True, repeat=1, label="", orc={}, **kw):
    from paper_2201_13007_amd import binding as B
    searched = base
    if dtype != "f32":
        searched = oracle.dequantize(*oracle.quantize(base, dtype), dtype)
    ix = B.Index(dev(base), dev(adj), 0, metric=metric, dtype=dtype)
    print(f"case: {label} n={base.shape[0]} d={base.shape[1]} nq={len(q) * repeat} L={L} M={M} {metric} {dtype}", flush=True)
    qs = dev(np.tile(q, (repeat, 1)))
    e = parity.oracle_search(searched, adj, 0, q, k, L, M, sync=sync, metric=metric, **orc)
    for _ in range(2):    # the second pass finds the workspace as the first left it
        r = ix.search(qs, k, L, M, stats=True, sync=sync, **orc, **kw)
        torch.cuda.synchronize()
        ids, d, st = r.ids.cpu().numpy(), r.dists.cpu().numpy(), r.stats.cpu().numpy()
        m = len(q)
        for x in (ids, d, st[:, :5]):    # every copy of the queries as the first
            np.testing.assert_array_equal(x, np.tile(x[:m], (repeat, 1)), err_msg=label)
        parity.compare((ids[:m], d[:m], st[:m]), e, exact, base=searched, queries=q, metric=metric, atol=1e-5,
                       label=label)


@pytest.mark.parametrize("nq", [5, MANY])
@pytest.mark.parametrize("d", [4, 8, 16, 20, 36, 64, 68, 100, 128, 132, 256, 260, 516, 960, 1024])
def test_vector_layouts(d, nq):
    g = np.random.default_rng(d)
    base = g.integers(-3, 4, (700, d)).astype(np.float32)
    q = g.integers(-3, 4, (5, d)).astype(np.float32)
    check(base, graph(700, 32, g), q, 10, 40, 2 if d % 8 else 1, "bsp", repeat=nq // 5, label="integers")


@pytest.mark.parametrize("nq", [6, MANY])
@pytest.mark.parametrize("dtype,metric", [("f32", "l2"), ("f32", "ip"), ("bf16", "ip"), ("fp8", "l2"), ("fp8", "ip")])
@pytest.mark.parametrize("d", [12, 96, 200])
def test_float_data(d, dtype, metric, nq):
    g = np.random.default_rng([d, 7])
    base = g.standard_normal((900, d)).astype(np.float32)
    q = g.standard_normal((5, d)).astype(np.float32)
    check(base, graph(900, 24, g), q, 10, 70, 1, "adaptive", metric, dtype, exact=False, repeat=nq // 5, label="floats")


@pytest.mark.parametrize("nq", [4, MANY])
@pytest.mark.parametrize("L", [1, 2, 63, 64, 65, 128, 129, 192, 193, 256, 257, 320, 321, 385, 449, 512, 513, 1023, 1024])
def test_queue_slots(L, nq):
    """Every number of slots per lane, its first and last L; from L = 512 on, the visited
    vertices outgrow the LDS sets of the many-queries form."""
    g = np.random.default_rng(L)
    n = 9000
    base = g.integers(0, 16, (n, 16)).astype(np.float32)
    q = g.integers(0, 16, (4, 16)).astype(np.float32)
    check(base, graph(n, 32, g), q, min(L, 20), L, 1 + L % 2, "bsp", repeat=nq // 4, label="slots")


@pytest.mark.parametrize("nq", [4, MANY])
@pytest.mark.parametrize("n", [3, 500, 70_000])
def test_visited_sets(n, nq):
    """Two distinct tags per set, tags of few bits, and sets that overflow by far."""
    g = np.random.default_rng(n)
    base = g.integers(0, 9, (n, 960 if n < 10_000 else 8)).astype(np.float32)
    q = g.integers(0, 9, (4, base.shape[1])).astype(np.float32)
    check(base, graph(n, 48, g), q, 2, 400 if n > 400 else 3, 1, "adaptive", repeat=nq // 4, label="visited",
          ws_hash_slots=1 << 16 if nq < 100 else 1 << 15)   # random rows: 48 new vertices a step


@pytest.mark.parametrize("nq", [60, MANY])
def test_integer_and_other_queries_together(nq):
    """Integer-valued vectors: integer queries in float32, the others in double, in one call."""
    g = np.random.default_rng(5)
    base = g.integers(0, 200, (2000, 64)).astype(np.float32)
    q = g.integers(0, 200, (20, 64)).astype(np.float32)
    q[::3] += 0.5
    q[1::7] = 1000.0
    check(base, graph(2000, 32, g), q, 10, 96, 1, "adaptive", exact=False, repeat=nq // 20, label="mixed")


@pytest.mark.parametrize("R", [20, 64])
@pytest.mark.parametrize("M", [2, 3, 4, 7, 16])
@pytest.mark.parametrize("L", [1, 2, 33, 64, 65, 200, 1024])
def test_several_workers_every_step(L, M, R):
    """Merges after every step: few and many new keys per step for the lanes that rank them,
    lists shorter than the workers, the staged start and all workers at once."""
    g = np.random.default_rng([L, M, R])
    n = 6000
    base = g.integers(0, 16, (n, 16)).astype(np.float32)
    q = g.integers(0, 16, (6, 16)).astype(np.float32)
    if R > 32 or M > 2:
        check(base, graph(n, R, g), q, min(L, 20), L, M, "bsp", repeat=1 + (M % 3), label="every step",
              ws_hash_slots=1 << 17)
        check(base, graph(n, R, g), q, min(L, 20), L, M, "bsp", label="every step, table in the workspace",
              ws_hash_slots=1 << 17, lds_hash_slots=-1)


@pytest.mark.parametrize("d", [4, 20, 96, 132, 260, 960])
@pytest.mark.parametrize("dtype,metric", [("f32", "l2"), ("bf16", "ip"), ("fp8", "l2")])
def test_several_workers_layouts(d, dtype, metric):
    g = np.random.default_rng([d, 11])
    base = g.standard_normal((900, d)).astype(np.float32)
    q = g.standard_normal((9, d)).astype(np.float32)
    check(base, graph(900, 32, g), q, 10, 70, 8, "bsp", metric, dtype, exact=False, label="workers, floats")
    if dtype == "f32":
        b, i = np.rint(4 * base), np.rint(4 * q)
        i[::2] += 0.5
        check(b, graph(900, 32, g), i, 10, 70, 5, "bsp", metric, dtype, exact=False, label="workers, integers")


def test_several_workers_limits():
    """The step limit, and visited sets that spill and fill up: flags and counters as before."""
    from paper_2201_13007_amd import binding as B
    g = np.random.default_rng(3)
    n = 70_000
    base = g.integers(0, 9, (n, 8)).astype(np.float32)
    adj = graph(n, 48, g)
    q = g.integers(0, 9, (4, 8)).astype(np.float32)
    ix = B.Index(dev(base), dev(adj), 0)
    for kw in ({"max_substeps": 5}, {"ws_hash_slots": 4096}, {"lds_hash_slots": 1024, "ws_hash_slots": 1 << 16}):
        a = ix.search(dev(q), 10, 300, 8, stats=True, sync="bsp", **kw)
        b = ix.search(dev(q), 10, 300, 8, stats=True, sync="static", static_I=1, **kw)   # the same schedule
        torch.cuda.synchronize()
        np.testing.assert_array_equal(a.ids.cpu().numpy(), b.ids.cpu().numpy())
        for name in FIELDS + ("flags",):
            np.testing.assert_array_equal(a.stat(name).cpu().numpy(), b.stat(name).cpu().numpy(), err_msg=f"{kw} {name}")
        assert a.stat("flags").cpu().numpy().any()


@pytest.mark.parametrize("sync,I", [("adaptive", 0), ("static", 0), ("static", 3)])
@pytest.mark.parametrize("M", [1, 2, 5, 16])
@pytest.mark.parametrize("L", [1, 30, 64, 128, 200, 513])
def test_several_workers_lazy(L, M, sync, I):
    """Merges now and then, or only at the end: own entries that outgrow their slots and are
    thinned out, entries that fall out of the local queue, more new entries than one round
    of a merge publishes."""
    g = np.random.default_rng([L, M, I])
    n = 6000
    base = g.integers(0, 16, (n, 16)).astype(np.float32)
    q = g.integers(0, 16, (6, 16)).astype(np.float32)
    for staged in (True, False):
        check(base, graph(n, 64, g), q, min(L, 20), L, M, sync, label=f"lazy {sync} {I} staged={staged}",
              ws_hash_slots=1 << 17, lds_hash_slots=4096, orc={"static_I": I, "rho": 0.7, "staged": staged})
