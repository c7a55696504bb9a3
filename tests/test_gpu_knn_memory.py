"""Exact kNN on a device with hardly any memory left: what the scan answers without any, it
still answers."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("d,k,integer", [(1024, 97, False), (1024, 256, False), (256, 129, True)])
def test_large_k_without_memory(d, k, integer):
    from paper_2201_13007_amd import binding as B
    n = 100_000 if d == 1024 else 400_000       # 0.4 GB of bf16 copies
    g = torch.Generator(device="cuda").manual_seed(d + k)
    x = torch.randint(0, 256, (n, d), generator=g, device="cuda").float()
    if not integer:
        x += 0.5
    qs = x[:3].clone()
    base, q = x.cpu().numpy(), qs.cpu().numpy()
    torch.cuda.empty_cache()
    print(f"case: n={n} d={d} k={k}", flush=True)
    fill = [torch.empty(torch.cuda.mem_get_info()[0] - (1 << 30), dtype=torch.uint8, device="cuda")]
    try:
        while len(fill) < 40:
            fill.append(torch.empty(96 << 20, dtype=torch.uint8, device="cuda"))
    except torch.OutOfMemoryError:
        del fill[1:3]
        torch.cuda.empty_cache()
    assert len(fill) < 40
    try:
        ids, dists, path = B.knn(x, qs, k, return_path=True)
        torch.cuda.synchronize()
    finally:
        del fill
        torch.cuda.empty_cache()
    assert path == "scan"
    eids, ed = oracle.knn(base, q, k)
    np.testing.assert_array_equal(ids.cpu().numpy(), eids)
    np.testing.assert_array_equal(dists.cpu().numpy(), ed)


def test_large_scratch_is_given_back():
    from paper_2201_13007_amd import binding as B
    x = torch.zeros((700_000, 1024), device="cuda")      # 2.9 GB of bf16 copies
    x[:, 0] = torch.arange(700_000, device="cuda") * 0.5
    B.knn(x[:1000].clone(), x[:2].clone(), 3)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    before = torch.cuda.memory_reserved()
    print("case: 700,000 x 1024", flush=True)
    ids, _ = B.knn(x, x[[5, 699_999]].clone(), 1)
    assert ids.flatten().tolist() == [5, 699_999]
    assert torch.cuda.memory_reserved() - before < (64 << 20)
