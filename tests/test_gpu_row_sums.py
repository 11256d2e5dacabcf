"""Bias gradients are summed in one fixed order: 256 partial sums of the columns
n = r mod 256 in order, then a tree, all in FP32.  Bitwise against the same sums in numpy, at
the edges of the unrolled loop, with odd rows and rows that start on 2 bytes only."""
import numpy as np
import pytest

from paper_2208_07129_amd import mfmv

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def ordered_sums(x):
    """x: M x N float32."""
    M, N = x.shape
    part = np.zeros((M, 256), np.float32)
    for n in range(0, N, 256):
        w = min(256, N - n)
        part[:, :w] += x[:, n:n + w]
    s = 128
    while s:
        part[:, :s] += part[:, s:2 * s]
        s //= 2
    return part[:, 0]


@pytest.mark.parametrize("M,N,pad,shift", [(3, 1, 7, 0), (8, 255, 1, 0), (7, 257, 1, 0),
                                           (5, 31 * 256 + 2, 0, 0), (4, 32 * 256 - 1, 1, 0),
                                           (4, 32 * 256, 0, 0), (6, 32768, 8, 0), (3, 40001, 1, 0),
                                           (4, 33000, 0, 3), (4, 33001, 0, 2), (2, 128000, 0, 0)])
@pytest.mark.parametrize("accumulate", [0, 1])
def test_row_sums_order(M, N, pad, shift, accumulate):
    gen = torch.Generator(device="cuda").manual_seed(N)
    buf = torch.randn(M * (N + pad) + shift, device="cuda", generator=gen).to(torch.bfloat16)
    X = buf[shift:].view(M, N + pad)
    out = torch.full((M,), 2.0, device="cuda")
    mfmv._check(mfmv.lib().mf_row_sums(M, N, X.data_ptr(), N + pad, out.data_ptr(), accumulate, None))
    torch.cuda.synchronize()
    want = ordered_sums(X[:, :N].float().cpu().numpy())
    if accumulate:
        want = np.float32(2.0) + want
    assert np.array_equal(out.cpu().numpy(), want)
