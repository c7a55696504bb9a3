"""Searches that merge after every step in small workspace tables: the visited set is bounded by
the tables' sizes and by nothing else (the static schedule with one step a merge is the same
search, and the oracle has no bound at all)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
FIELDS = ("global_steps", "substeps", "expansions", "dist_comps", "merges")


# many ids (two tags or none to a set in LDS) and short lists (few sets): hundreds of vertices
# find their set full, more than the smallest workspace tables hold
@pytest.mark.parametrize("n,R,L,M,lds,ws", [
    (1 << 20, 16, 32, 3, 0, 128), (1 << 20, 16, 64, 4, 0, 128), (1 << 20, 16, 64, 4, 0, 256),
    (1 << 20, 16, 40, 8, 0, 256), (1 << 20, 32, 32, 5, 8192, 512), (70_000, 64, 32, 16, 8192, 2048),
    (1 << 20, 24, 32, 2, 4096, 128), (3 << 19, 64, 48, 16, 16384, 2048), (1 << 20, 16, 64, 4, 0, 4096)])
@pytest.mark.parametrize("staged", [True, False])
def test_every_step_small_tables(n, R, L, M, lds, ws, staged):
    from paper_2201_13007_amd import binding as B
    g = np.random.default_rng([n, R, L, M])
    base = g.integers(0, 50, (n, 8)).astype(np.float32)
    adj = g.integers(0, n, (n, R)).astype(np.int32)
    q = g.integers(0, 50, (7, 8)).astype(np.float32)
    ix = B.Index(torch.from_numpy(base).cuda(), torch.from_numpy(adj).cuda(), 0)
    print(f"case: n={n} R={R} L={L} M={M} lds_hash_slots={lds} ws_hash_slots={ws} staged={staged}", flush=True)
    kw = dict(lds_hash_slots=lds, ws_hash_slots=ws, staged=staged)
    qs = torch.from_numpy(q).cuda()
    want = ix.search(qs, 10, L, M, stats=True, sync="static", static_I=1, **kw)
    e = oracle.speedann(base, adj, 0, q, 10, L, M, sync="bsp", staged=staged)
    for _ in range(2):    # the second pass finds the workspace as the first left it
        got = ix.search(qs, 10, L, M, stats=True, sync="bsp", **kw)
        torch.cuda.synchronize()
        assert torch.equal(got.ids, want.ids) and torch.equal(got.dists, want.dists)
        for name in FIELDS + ("flags",):
            np.testing.assert_array_equal(got.stat(name).cpu().numpy(), want.stat(name).cpu().numpy(), err_msg=name)
        whole = (got.stat("flags").cpu().numpy() & B.QFLAG_CAPACITY) == 0
        np.testing.assert_array_equal(got.ids.cpu().numpy()[whole], e[0][whole])
        np.testing.assert_array_equal(got.stat("dist_comps").cpu().numpy()[whole], e[2]["dist_comps"][whole])
