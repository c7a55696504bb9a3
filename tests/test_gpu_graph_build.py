"""Reverse edges and repair on the device, at the edges of their lists, rows and groups,
against the oracle (bit for bit)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle


@pytest.fixture(scope="module")
def B():
    from paper_2201_13007_amd import binding
    binding.lib()
    return binding


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def random_rows(rng, n, R, fill, targets):
    """n rows of up to `fill` of R distinct out-neighbours drawn from `targets`, -1 padded."""
    adj = np.full((n, R), -1, np.int32)
    for v in range(n):
        t = rng.choice(targets, size=min(fill, len(targets)), replace=False)
        t = t[t != v][: rng.integers(0, fill + 1)]
        adj[v, : len(t)] = t
    return adj


# in-degrees from none to thousands (lists of one, several and many chunks of 64), rows with
# one to all slots free, equal distances, neighbours that are in the row already
@pytest.mark.parametrize("n,R,fill,ntarget", [(2, 1, 1, 2), (300, 4, 3, 300), (3000, 32, 8, 3000), (3000, 32, 8, 40),
                                              (2500, 64, 20, 2500), (2500, 64, 30, 70), (4100, 16, 2, 3)])
@pytest.mark.parametrize("metric", ["l2", "ip"])
def test_reverse_edges_lists(B, n, R, fill, ntarget, metric):
    rng = np.random.default_rng(n + R + ntarget)
    base = rng.integers(-3, 4, size=(n, 8)).astype(np.float32)
    adj = random_rows(rng, n, R, fill, rng.choice(n, size=min(ntarget, n), replace=False))
    # some back edges: the source of an in-edge is in the row already
    for v in range(0, n, 3):
        u = adj[v, 0]
        if u >= 0 and u != v:
            free = np.flatnonzero(adj[u] < 0)
            if len(free) > R // 2 and v not in adj[u]:
                adj[u, free[0]] = v
    want = adj.copy()
    wa = oracle.reverse_edges(base, want, metric=metric)
    g = dev(adj)
    print(f"case: reverse edges n={n} R={R} targets={ntarget} {metric} added={wa}", flush=True)
    assert B.reverse_edges(dev(base), g, metric=metric) == wa
    np.testing.assert_array_equal(g.cpu().numpy(), want)


# groups: one; a few; 65; one large and many single vertices; more than the link kernel sorts
# (4096: links on the host)
@pytest.mark.parametrize("kind,n", [("one", 700), ("three", 900), ("65", 1300), ("lonely", 1500), ("pairs", 9000)])
@pytest.mark.parametrize("metric,d,R", [("l2", 68, 16), ("ip", 8, 32)])
def test_repair_groups(B, kind, n, metric, d, R):
    rng = np.random.default_rng(n + d)
    base = rng.standard_normal((n, d)).astype(np.float32)
    groups = {"one": 1, "three": 3, "65": 65, "lonely": 200, "pairs": n // 2}[kind]
    if kind == "lonely":
        label = np.where(np.arange(n) % 7 == 0, 1 + np.arange(n) // 7, 0)
    elif kind == "pairs":
        label = np.arange(n) // 2
    else:
        label = np.arange(n) % groups
    adj = np.full((n, R), -1, np.int32)
    for c in np.unique(label):
        m = np.flatnonzero(label == c)
        if len(m) > 1:
            nxt = np.roll(m, -1)
            adj[m, 0] = nxt
            for v in m:
                t = rng.choice(m, size=min(3, len(m)), replace=False)
                t = [int(u) for u in t if u != v and u not in adj[v]]
                adj[v, 1 : 1 + len(t)] = t
    # some vertices nobody points to
    if kind in ("one", "three"):
        gone = rng.choice(n, size=40, replace=False)
        adj[np.isin(adj, gone)] = -1
        for v in range(n):
            row = adj[v][adj[v] >= 0]
            adj[v] = -1
            adj[v, : len(row)] = row
    entry = oracle.medoid(base)
    for keep, hubs, hub_keep in ((1, 5, 2), (2, 1, 1)):
        want = adj.copy()
        wb, wc = oracle.repair(base, want, entry, keep_local=keep, hubs=hubs, hub_keep_local=hub_keep, metric=metric)
        g = dev(adj)
        print(f"case: repair {kind} n={n} {metric} keep={keep} hubs={hubs} bridges={wb} comps={wc}", flush=True)
        assert B.repair(dev(base), g, entry, keep_local=keep, metric=metric, hubs=hubs, hub_keep_local=hub_keep) == (wb, wc)
        np.testing.assert_array_equal(g.cpu().numpy(), want)
