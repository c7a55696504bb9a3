"""An untuned batch runs its classes side by side on streams of its own: the same results as
one after the other, from several threads and streams at once, and under capture."""
import threading

import numpy as np
import pytest

from paper_2201_13007_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_default_plan_streams_threads_capture():
    from paper_2201_13007_amd import binding as B
    w = synth.sift_like(n=4000, nq=90)
    base = torch.from_numpy(w.base).cuda()
    adj, entry, _ = B.build_graph(base, 32, 24)
    ix = B.Index(base, adj, entry)
    g = np.random.default_rng(2)
    L = g.integers(20, 400, 90).astype(np.int32)
    M = g.choice(np.array([1, 2, 4, 8], np.int32), 90)
    k = np.full(90, 10, np.int32)
    q = torch.from_numpy(w.queries).cuda()
    one = B.Batch(ix, L, k, M)
    one.set_config(1)
    want = one.run(q, stats=True)
    torch.cuda.synchronize()

    def same(r, order=slice(None)):
        assert torch.equal(r.ids, want.ids[order]) and torch.equal(r.dists, want.dists[order])

    b = B.Batch(ix, L, k, M)
    assert b.classes() > 4
    print("case: batch default plan, repeated", flush=True)
    for _ in range(3):
        r = b.run(q, stats=True)
        torch.cuda.synchronize()
        same(r)
        assert torch.equal(r.stats[:, :5], want.stats[:, :5])
    assert not b.ws[b.ws.numel() - 4096:].any()   # the last class's regions are zero again

    print("case: one batch from three threads with streams and workspaces of their own", flush=True)
    out, keep = {}, []

    def work(i):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            mine = B.Batch(ix, L, k, M) if i else b
            keep.append(mine)
            for _ in range(5):
                out[i] = mine.run(q)
        s.synchronize()

    ts = [threading.Thread(target=work, args=(i,)) for i in range(3)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    for i in range(3):
        same(out[i])

    print("case: captured and replayed", flush=True)
    ids, dists, _ = b.outputs()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        b.run(q, out=(ids, dists, None))
    torch.cuda.current_stream().wait_stream(s)
    gr = torch.cuda.CUDAGraph()
    with torch.cuda.graph(gr):
        b.run(q, out=(ids, dists, None))
    for _ in range(3):
        ids.fill_(-7)
        gr.replay()
        torch.cuda.synchronize()
        same(B.SearchResult(ids, dists, None))
        same(b.run(q))                       # eager work between the replays
    del b
