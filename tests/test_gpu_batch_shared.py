"""One plan run by several threads at once, each on a stream, workspace, queries and outputs of
its own: they share the plan's internal streams and events."""
import threading

import numpy as np
import pytest

from paper_2201_13007_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_one_plan_many_threads():
    from paper_2201_13007_amd import binding as B
    w = synth.sift_like(n=4000, nq=90)
    base = torch.from_numpy(w.base).cuda()
    adj, entry, _ = B.build_graph(base, 32, 24)
    ix = B.Index(base, adj, entry)
    g = np.random.default_rng(2)
    L = g.integers(20, 400, 90).astype(np.int32)
    M = g.choice(np.array([1, 2, 4, 8], np.int32), 90)
    b = B.Batch(ix, L, np.full(90, 10, np.int32), M)
    lib = B.lib()
    n_threads, rounds = 4, 25
    jobs = []
    for i in range(n_threads):
        q = torch.from_numpy(np.roll(w.queries, 7 * i + 1, axis=0).copy()).cuda()
        ws = torch.zeros_like(b.ws)
        s = torch.cuda.Stream()
        torch.cuda.synchronize()
        assert lib.sa_batch_upload(b._h, ws.data_ptr(), ws.numel(), s.cuda_stream) == 0
        s.synchronize()
        jobs.append((q, ws, s, [b.outputs() for _ in range(rounds)]))
    one = B.Batch(ix, L, np.full(90, 10, np.int32), M)
    one.set_config(1)
    want = [one.run(q) for q, *_ in jobs]
    torch.cuda.synchronize()
    rcs = [[] for _ in range(n_threads)]
    start = threading.Barrier(n_threads)

    def work(i):
        q, ws, s, outs = jobs[i]
        start.wait()
        for ids, dists, _ in outs:
            rcs[i].append(lib.sa_batch_run(b._h, q.data_ptr(), q.stride(0), ids.data_ptr(), dists.data_ptr(),
                                           ids.stride(0), None, ws.data_ptr(), ws.numel(), s.cuda_stream))
        s.synchronize()

    print(f"case: one plan from {n_threads} threads", flush=True)
    ts = [threading.Thread(target=work, args=(i,)) for i in range(n_threads)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    torch.cuda.synchronize()
    for i, (_, ws, _, outs) in enumerate(jobs):
        assert rcs[i] == [0] * rounds
        for ids, dists, _ in outs:
            assert torch.equal(ids, want[i].ids) and torch.equal(dists, want[i].dists)
