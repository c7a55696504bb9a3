"""knn on streams of other libraries: any object that has a stream's handle."""
from types import SimpleNamespace

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_stream_objects():
    from paper_2201_13007_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(4)
    x = torch.randn(5000, 64, generator=g, device="cuda")
    q = torch.randn(30, 64, generator=g, device="cuda")
    want = B.knn(x, q, 10)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    for stream in (s, SimpleNamespace(cuda_stream=s.cuda_stream), SimpleNamespace(cuda_stream=0)):
        print(f"case: {type(stream).__name__}", flush=True)
        for path in ("auto", "scan"):
            ids, d = B.knn(x, q, 10, stream=stream, path=path)
            assert torch.equal(ids, want[0]) and torch.equal(d, want[1])
