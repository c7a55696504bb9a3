"""Repairs that fail, and graphs of more rows than a launch takes work items at one wavefront
a row."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_failed_repair_leaves_the_rows():
    """Two components of full rows, one vertex of the second out of reach: its representative's
    and the first one's rows get links, then no reachable vertex has a free slot."""
    from paper_2201_13007_amd import binding as B
    base = np.zeros((7, 4), np.float32)
    base[:, 0] = [5, 0, 1, 50, 60, 90, 2]          # medoids: vertex 2 (rows 0, 1, 2, 6) and 4
    adj = np.array([[1, 2], [0, 2], [0, 1], [4, 4], [3, 3], [4, -1], [0, 1]], np.int32)
    adj[2] = [6, 0]
    lost = adj.copy()
    g = torch.from_numpy(adj).cuda()
    print("case: repair without a free slot", flush=True)
    with pytest.raises(RuntimeError, match="free slot"):
        B.repair(torch.from_numpy(base).cuda(), g, 0, keep_local=1, hubs=1, hub_keep_local=2)
    np.testing.assert_array_equal(g.cpu().numpy(), lost)
    # with room it succeeds, and is the oracle's
    wide = np.full((7, 4), -1, np.int32)
    wide[:, :2] = adj
    want = wide.copy()
    b, c = oracle.repair(base, want, 0, keep_local=1, hubs=1, hub_keep_local=2)
    g = torch.from_numpy(wide).cuda()
    assert B.repair(torch.from_numpy(base).cuda(), g, 0, keep_local=1, hubs=1, hub_keep_local=2) == (b, c)
    np.testing.assert_array_equal(g.cpu().numpy(), want)


def test_more_rows_than_a_launch_has_wavefronts():
    """2^26 + 1000 rows of 64 entries: a tree, every vertex linked to its 64 children.  The
    vertices with room get their parent; then all are one component within reach."""
    from paper_2201_13007_amd import binding as B
    n, R = (1 << 26) + 1000, 64
    base = torch.zeros((n, 4), device="cuda")
    base[:, 0] = torch.arange(n, device="cuda") % 1000
    adj = torch.empty((n, R), dtype=torch.int32, device="cuda")
    for r0 in range(0, n, 1 << 23):
        v = torch.arange(r0, min(n, r0 + (1 << 23)), device="cuda")
        c = v[:, None] * R + 1 + torch.arange(R, device="cuda")
        adj[r0:r0 + len(v)] = torch.where(c < n, c, -1).int()
        del c
    inner = (n - 1) // R      # vertices whose row is full; the next may have some children
    some = n - 1 - inner * R
    print(f"case: tree of {n} rows", flush=True)
    assert B.reverse_edges(base, adj) == n - inner
    v = torch.arange(inner + 1, n, device="cuda")
    assert bool((adj[inner + 1:, 0] == ((v - 1) // R).int()).all()) and bool((adj[inner + 1:, 1:] == -1).all())
    assert adj[inner, some].item() == (inner - 1) // R
    info = B.repair(base, adj, 0)
    assert tuple(info) == (0, 1)


# 4,096 rows of 32 are the largest whose components and reachability come from the host
@pytest.mark.parametrize("n", [4096, 4097, 7000])
@pytest.mark.parametrize("groups,gone", [(1, 0), (1, 60), (3, 25), (90, 200)])
@pytest.mark.parametrize("metric", ["l2", "ip"])
def test_repair_host_and_device(n, groups, gone, metric):
    from paper_2201_13007_amd import binding as B
    R = 32
    rng = np.random.default_rng([n, groups, gone])
    base = rng.standard_normal((n, 12)).astype(np.float32)
    label = rng.integers(0, groups, n)
    label[:groups] = np.arange(groups)
    adj = np.full((n, R), -1, np.int32)
    for c in range(groups):
        m = np.flatnonzero(label == c)
        if len(m) > 1:
            adj[m, 0] = np.roll(m, -1)
            adj[m, 1] = np.roll(m, -len(m) // 2)
            adj[m, 2] = rng.permutation(m)
    adj[np.isin(adj, rng.choice(n, gone, replace=False))] = -1    # nobody points there
    adj = np.take_along_axis(adj, np.argsort(adj < 0, axis=1, kind="stable"), axis=1)
    entry = oracle.medoid(base)
    want = adj.copy()
    wb, wc = oracle.repair(base, want, entry, keep_local=1, hubs=9, hub_keep_local=2, metric=metric)
    g = torch.from_numpy(adj).cuda()
    print(f"case: n={n} groups={groups} gone={gone} {metric} bridges={wb} components={wc}", flush=True)
    assert B.repair(torch.from_numpy(base).cuda(), g, entry, keep_local=1, metric=metric, hubs=9, hub_keep_local=2) == (wb, wc)
    np.testing.assert_array_equal(g.cpu().numpy(), want)


# a prefix sum of up to 2,048 counts is one launch
@pytest.mark.parametrize("n", [1, 2047, 2048, 2049, 6000])
def test_reverse_edges_chunks(n):
    from paper_2201_13007_amd import binding as B
    rng = np.random.default_rng(n)
    base = rng.integers(-3, 4, (n, 4)).astype(np.float32)
    adj = rng.integers(0, n, (n, 6)).astype(np.int32)
    adj[:, 2:] = -1
    adj[:, 1] = np.where(adj[:, 1] == adj[:, 0], -1, adj[:, 1])
    want = adj.copy()
    wa = oracle.reverse_edges(base, want)
    g = torch.from_numpy(adj).cuda()
    print(f"case: reverse edges n={n} added={wa}", flush=True)
    assert B.reverse_edges(torch.from_numpy(base).cuda(), g) == wa
    np.testing.assert_array_equal(g.cpu().numpy(), want)
