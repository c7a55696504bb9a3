"""The framework's work as measured cases: graph searches from one query to ten thousand,
mixed batches, exact kNN, graph construction and reduced-precision encoding, over data
shaped like the workloads of this repository (synth.py), generated on the GPU.

Families (the "path" of a case):
  search    Index.search over a graph built from the case's own data: one query for latency,
            a few, or a whole batch; float32 (integer-valued or not), bf16 and fp8 storage,
            with and without the exact re-rank; one to sixteen walkers
  batch     Batch.run: queries with their own (L, k, M) in one plan
  knn       exact k nearest neighbours (ground truth): integer-valued and float data
  build     build_graph: medoid, exact candidates, pruning, reverse edges, repair
  quantize  the reduced-precision copy of a set of vectors
"""
import math

import numpy as np
import torch

from paper_2201_13007_amd import binding as B


def _search(name, data, n, d, nq, k, L, M, sync, dtype="f32", rerank=0, order="none"):
    return {"name": name, "path": "search", "data": data, "n": n, "d": d, "nq": nq, "k": k, "L": L, "M": M,
            "sync": sync, "dtype": dtype, "rerank": rerank, "order": order}


def listed():
    return [
        # one interactive request on the 1M SIFT-shaped index: sixteen walkers for latency
        _search("search_one_m16", "sift", 1_000_000, 128, 1, 10, 176, 16, "bsp"),
        # a handful of requests that arrived together, the default (adaptive) schedule
        _search("search_33_m8", "sift", 200_001, 128, 33, 10, 272, 8, "adaptive"),
        # a small call over low-dimensional float data, one walker, every option at its default
        _search("search_tiny_100", "tiny", 10_000, 32, 100, 10, 64, 1, "adaptive"),
        # the throughput point: ten thousand queries, two walkers merging every step, the
        # index renumbered breadth first
        _search("search_10k_m2", "sift", 1_000_000, 128, 10_000, 10, 192, 2, "bsp", order="bfs"),
        # the same use on bf16 embeddings with the whole final list re-ranked
        _search("search_10k_bf16", "deep", 1_000_000, 96, 10_000, 10, 112, 2, "bsp", "bf16", -1),
        # a serving micro-batch at a high recall target: fp8 codes, one walker, re-ranked
        _search("search_1k_fp8", "deep", 200_000, 96, 1_001, 100, 512, 1, "adaptive", "fp8", -1),
        # mixed requests over wide descriptors, planned as one batch
        {"name": "batch_mixed_d960", "path": "batch", "data": "gist", "n": 100_000, "d": 960, "nq": 2_000},
        # ground truth for a benchmark set: integer-valued descriptors
        {"name": "knn_int_10k", "path": "knn", "data": "sift", "n": 1_000_000, "d": 128, "nq": 10_000, "k": 10},
        # ground truth at k = 100 for a smaller set of float queries, inner product
        {"name": "knn_float_k100", "path": "knn", "data": "deep", "n": 1_000_000, "d": 96, "nq": 1_000, "k": 100},
        # wide float descriptors, candidate-list sized k
        {"name": "knn_wide_2k", "path": "knn", "data": "gist", "n": 200_000, "d": 960, "nq": 2_000, "k": 64},
        # an index built from scratch
        {"name": "build_150k", "path": "build", "data": "sift", "n": 150_001, "d": 128, "R": 32},
        # the fp8 copy of a vector set
        {"name": "quantize_fp8_1m", "path": "quantize", "data": "deep", "n": 1_000_000, "d": 96, "dtype": "fp8"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_DIMS = {"tiny": (16, 32, 50), "sift": (64, 100, 128), "deep": (64, 96, 200), "gist": (384, 960)}


def draw(rng):
    path = rng.choice(["search"] * 5 + ["knn"] * 3 + ["batch", "build", "quantize"])
    if path == "search":
        data = rng.choice(["tiny", "sift", "sift", "deep", "deep"])
        dtype = rng.choice(["f32", "bf16", "fp8"]) if data == "deep" else "f32"
        M, sync = rng.choice([(1, "adaptive"), (2, "bsp"), (4, "adaptive"), (8, "bsp"), (16, "bsp"), (16, "adaptive")])
        L = _log(rng, 32, 768)
        nq = min(_log(rng, 1, 10_000), 1_500_000 // L)
        if M > 2:
            nq = min(nq, 200_000 // L)
        n = _log(rng, 5_000, 50_000) if data == "tiny" else _log(rng, 20_000, 500_000)
        return _search("", data, n, rng.choice(_DIMS[data]), nq, min(L, rng.choice([1, 10, 100])), L, M, sync, dtype,
                       rng.choice([0, -1]) if dtype != "f32" else 0, rng.choice(["none", "bfs"]))
    if path == "batch":
        return {"path": path, "data": "gist", "n": _log(rng, 20_000, 100_000), "d": rng.choice(_DIMS["gist"]),
                "nq": _log(rng, 100, 2_000)}
    if path == "knn":
        data = rng.choice(["tiny", "sift", "deep", "gist"])
        return {"path": path, "data": data, "n": _log(rng, 20_000, 200_000 if data == "gist" else 1_000_000),
                "d": rng.choice(_DIMS[data]), "nq": _log(rng, 1, 2_000 if data == "gist" else 10_000),
                "k": rng.choice([1, 10, 64, 100])}
    if path == "build":
        data = rng.choice(["sift", "deep"])
        return {"path": path, "data": data, "n": _log(rng, 20_000, 150_000), "d": rng.choice(_DIMS[data]),
                "R": rng.choice([24, 32, 48])}
    return {"path": path, "data": rng.choice(["deep", "gist"]), "n": _log(rng, 1_000, 200_000),
            "d": rng.choice([64, 96, 100, 200, 384]), "dtype": rng.choice(["bf16", "fp8"])}


def _vectors(case, seed):
    """(base, queries): the shapes and value distributions of synth.py's workloads."""
    n, nq, d, kind = case["n"], case.get("nq", 0), case["d"], case["data"]
    g = torch.Generator(device="cuda").manual_seed(seed * 1009 + 17)

    def rand(*s):
        return torch.rand(*s, generator=g, device="cuda")

    if kind == "tiny":
        x = rand(n + nq, d)
        return x[:n].clone(), x[n:].clone()
    ncomp = {"sift": 256, "deep": 512, "gist": 128}[kind]
    means = torch.randn(ncomp, d, generator=g, device="cuda") if kind == "deep" else rand(ncomp, d)
    label = torch.randint(0, ncomp, (n + nq,), generator=g, device="cuda")
    noise = torch.randn(n + nq, d, generator=g, device="cuda")
    if kind == "sift":
        x = (255.0 * means[label] + 20.0 * noise).round().clamp(0, 255)
    elif kind == "gist":
        x = means[label] + 0.1 * noise
    else:
        sd = torch.arange(1, d + 1, device="cuda", dtype=torch.float32).rsqrt()
        x = (means[label] + noise) * sd
        x = x / x.norm(dim=1, keepdim=True)
    return x[:n].clone(), x[n:].clone()


def _metric(case):
    return "ip" if case["data"] == "deep" else "l2"


def _mixed(case, seed):
    """Per-query (L, k, M) of a mixed batch: L log-uniform in [32, 1024] raised to k."""
    g = np.random.default_rng([2201, 13007, 4, seed])
    nq = case["nq"]
    k = g.choice(np.array([1, 10, 100], np.int32), size=nq)
    L = np.maximum(np.rint(np.exp(g.uniform(np.log(32.0), np.log(1024.0), size=nq))).astype(np.int32), k)
    return L, k, g.choice(np.array([1, 4, 8], np.int32), size=nq)


def prepare(case, seed):
    base, queries = _vectors(case, seed)
    st = {"case": case, "base": base, "queries": queries}
    path = case["path"]
    if path in ("search", "batch"):
        m = _metric(case)
        if case["data"] == "tiny":
            adj, entry, _ = B.build_graph(base, 16, 16, prune_mode="knn", do_repair=False, metric=m)
        else:
            adj, entry, _ = B.build_graph(base, 64, 32, metric=m)
        perm = None
        if case.get("order") == "bfs":
            base, adj, entry, perm = B.reorder(base, adj, entry, "bfs")
        st["index"] = B.Index(base, adj, entry, m, dtype=case.get("dtype", "f32"), id_map=perm)
    if path == "search":
        st["params"] = B.make_params(sync=case["sync"], rerank=case["rerank"])
    if path == "batch":
        st["batch"] = B.Batch(st["index"], *_mixed(case, seed))
    torch.cuda.synchronize()
    return st


def run(st):
    case = st["case"]
    path = case["path"]
    if path == "search":
        r = st["index"].search(st["queries"], case["k"], case["L"], case["M"], params=st["params"])
        return r.ids, r.dists
    if path == "batch":
        r = st["batch"].run(st["queries"])
        return r.ids, r.dists
    if path == "knn":
        return B.knn(st["base"], st["queries"], case["k"], metric=_metric(case))
    if path == "build":
        adj, entry, info = B.build_graph(st["base"], 64, case["R"], metric=_metric(case))
        return adj, entry, info["bridges"], info["components"]
    return B.quantize(st["base"], case["dtype"])


def work(case):
    n, d, path = case["n"], case["d"], case["path"]
    if path in ("search", "batch"):
        # a search with queue size L computes some 10 L distances and expands about L vertices
        # (counters of the 1M-row workloads); each distance reads one stored vector
        size = {"f32": 4, "bf16": 2, "fp8": 1}[case.get("dtype", "f32")]
        Ls = [case["L"]] * case["nq"] if path == "search" else [int(v) for v in _mixed(case, 0)[0]]
        k = case.get("k", 37)
        dist = sum(min(n, 10 * L) for L in Ls)
        rr = sum(Ls) * d * 4 if case.get("rerank", 0) else 0
        return {"bytes": dist * d * size + sum(Ls) * 32 * 4 + rr + len(Ls) * (4 * d + 8 * k), "flops": 3 * d * dist}
    if path == "knn":
        nq, k = case["nq"], case["k"]
        return {"bytes": 4 * d * (n + nq) + 8 * nq * k, "flops": 2 * d * n * nq}
    if path == "build":
        return {"bytes": 4 * d * n + 4 * n * case["R"], "flops": 2 * d * n * n}
    return {"bytes": n * (4 * d + (2 if case["dtype"] == "bf16" else 1) * d + 4), "flops": n * d}


def exact(case, seed):
    """kNN: ids and 64-bit distances by brute force, ordered by (distance rounded to float32,
    id).  Quantize: the fp8 scales.  A search's or a build's answer is defined by the graph
    that the framework builds, so there is no such value for it."""
    if case["path"] == "quantize":
        base = _vectors(case, seed)[0].double()
        if case["dtype"] == "bf16":
            return None, torch.ones(case["n"], dtype=torch.float64, device="cuda")
        amax = base.abs().amax(dim=1)
        return None, torch.where(amax > 0, amax / 448.0, torch.ones_like(amax))
    if case["path"] != "knn":
        return None
    base, queries = _vectors(case, seed)
    k, l2 = case["k"], _metric(case) == "l2"
    ids, dists = [], []
    for q0 in range(0, case["nq"], 1000):
        q = queries[q0:q0 + 1000].double()
        best_key = best_d = None
        for x0 in range(0, case["n"], 200_000):
            x = base[x0:x0 + 200_000].double()
            dot = q @ x.T
            dd = (q * q).sum(1, keepdim=True) + (x * x).sum(1) - 2 * dot if l2 else -dot
            b = (dd.float() + 0.0).view(torch.int32).long()   # order of floats as integers, -0 as +0
            key = torch.where(b >= 0, b, -(b & 0x7FFFFFFF)) * (1 << 32) + torch.arange(x0, x0 + x.shape[0], device="cuda")
            if best_key is not None:
                key, dd = torch.cat([best_key, key], 1), torch.cat([best_d, dd], 1)
            best_key, at = key.topk(min(k, key.shape[1]), dim=1, largest=False, sorted=True)
            best_d = dd.gather(1, at)
        ids.append((best_key & 0xFFFFFFFF).int())
        dists.append(best_d)
    return torch.cat(ids), torch.cat(dists)
