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
