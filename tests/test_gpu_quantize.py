"""Quantization at the edges of its row layouts: 8 to 64 lanes per row, up to four and up to
sixteen chunks a lane, padded code rows, and the values its rounding can go wrong on."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("d,pad", [(4, 0), (36, 0), (96, 4), (128, 8), (132, 0), (260, 4), (512, 0), (516, 0),
                                   (1024, 0), (1028, 4), (4096, 0)])
def test_codes(dtype, d, pad):
    from paper_2201_13007_amd import binding as B
    g = np.random.default_rng([d, pad])
    n = 67
    x = g.standard_normal((n, d)).astype(np.float32)
    x *= np.exp2(g.integers(-20, 20, (n, d))).astype(np.float32)   # codes down to the smallest
    x[0] = 0.0
    x[1, ::2] = -0.0
    x[2] *= np.float32(2.0 ** -90)    # scales outside the range of the reciprocal form
    x[3] *= np.float32(2.0 ** 70)
    x[4] = np.float32(2.0 ** -140)
    # quotients exactly on and next to the boundaries between codes: amax 448 makes the scale 1
    # (or 2^-30)
    mid = np.float32([0.5 * 2.0 ** -9, 1.5 * 2.0 ** -9, 17.0 / 16, 1.1875, 464.0 / 2, 29 * 8.0])
    for r, f in ((5, 1.0), (6, 2.0 ** -30)):
        vals = np.concatenate([mid, np.nextafter(mid, np.float32(0)), np.nextafter(mid, np.float32(1e9)), -mid])
        x[r] = np.resize(vals, d) * np.float32(f)
        x[r, 0] = np.float32(448.0 * f)
    print(f"case: quantize {dtype} {n}x{d} pad {pad}", flush=True)
    xd = torch.from_numpy(x).cuda()
    codes = torch.full((n, d + pad), 0x55, dtype=torch.int16 if dtype == "bf16" else torch.uint8, device="cuda")
    scale = torch.empty(n, dtype=torch.float32, device="cuda")
    B._check(B.lib().sa_quantize(xd.data_ptr(), n, d, d, B.DTYPES[dtype], codes.data_ptr(), d + pad,
                                 scale.data_ptr(), B._stream(None)), "sa_quantize")
    torch.cuda.synchronize()
    ec, es = oracle.quantize(x, dtype)
    got = codes.cpu().numpy().view(ec.dtype)
    np.testing.assert_array_equal(scale.cpu().numpy(), es)
    np.testing.assert_array_equal(got[:, :d], ec)
    assert not got[:, d:].any()


def test_fp8_nan_and_infinity():
    """A NaN saturates with its sign; an infinite coordinate makes the scale infinite, its own
    code saturate and every finite code zero."""
    from paper_2201_13007_amd import binding as B
    x = np.ones((2, 8), np.float32)
    x[0, 3], x[0, 4], x[0, 5] = np.float32(np.nan), -np.float32(np.nan), -0.25
    x[1, 2], x[1, 6] = np.inf, -1.0
    codes, scale = B.quantize(torch.from_numpy(x).cuda(), "fp8")
    torch.cuda.synchronize()
    c = codes.cpu().numpy()
    assert scale.cpu().numpy()[0] == np.float32(1.0) / np.float32(448.0) and np.isinf(scale.cpu().numpy()[1])
    assert c[0].tolist() == [0x7E, 0x7E, 0x7E, 0x7E, 0xFE, 0xEE, 0x7E, 0x7E]
    assert c[1].tolist() == [0, 0, 0x7E, 0, 0, 0, 0x80, 0]
