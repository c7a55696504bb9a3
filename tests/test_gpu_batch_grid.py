"""The grid of a batch's persistent form depends on the workgroup size: two classes of the same
kernel and LDS size, five and four wavefronts to a workgroup."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def most_at_once(times):
    """times: [n][2], start and end."""
    ev = sorted([(t, 1) for t in times[:, 0]] + [(t, -1) for t in times[:, 1]])
    return int(np.max(np.cumsum([d for _, d in ev])))


def test_grid_by_workgroup_size():
    from paper_2201_13007_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(3)
    n, d = 4000, 1024
    base = torch.randn(n, d, generator=g, device="cuda")
    adj = torch.randint(0, n, (n, 32), generator=g, device="cuda", dtype=torch.int32)
    ix = B.Index(base, adj, 0, metric="ip", dtype="bf16")
    most = {}
    for M, L in ((5, 32), (4, 64), (4, 100)):
        nq = 3000
        q = torch.randn(nq, d, generator=g, device="cuda")
        b = B.Batch(ix, np.full(nq, L, np.int32), np.full(nq, 5, np.int32), np.full(nq, M, np.int32),
                    params=B.make_params(sync="bsp"))
        assert b.classes() == 1
        want = b.run(q)
        torch.cuda.synchronize()
        b.set_class(0, 0, True)
        print(f"case: M={M} L={L}", flush=True)
        r = b.run(q, stats=True)
        torch.cuda.synchronize()
        assert torch.equal(r.ids, want.ids)
        most[M, L] = most_at_once(r.times().cpu().numpy())
    print(f"at once: {most}", flush=True)
    assert most[4, 64] > 0.9 * most[4, 100], most    # nearly the same kernel, of another LDS size
