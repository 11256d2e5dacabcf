"""A split K range of the BF16 product is cut where the caller says: ceil(K / kchunk) pieces,
each adding its FP32 sum to an element once.  One piece therefore repeats to the bit and
equals the undivided product, and two give the FP32 sum of the two products, whichever
arrives first."""
import pytest

from paper_2208_07129_amd import mlp

from test_gpu_gemm_forms import random_bf16

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def product(A, B, K, ldk, kchunk=0, atomic=True):
    M, N = A.shape[0], B.shape[0]
    out = torch.zeros(M, N, device="cuda")
    mlp.CellMLP._gemm(M, N, K, False, True, A, ldk, B, ldk, kchunk=kchunk, out_f32=out, ld_f32=N,
                      atomic=atomic)
    return out


@pytest.mark.parametrize("M,N,K,kchunk", [(8, 8, 40000, 40000), (64, 96, 8192, 8192),
                                          (256, 344, 8200, 16384), (344, 600, 1032, 1 << 20)])
def test_one_piece(M, N, K, kchunk):
    A = random_bf16(M, K, seed=1).view(torch.int16)
    B = random_bf16(N, K, seed=2).view(torch.int16)
    whole = product(A, B, K, K, atomic=False)
    for _ in range(3):
        assert torch.equal(product(A, B, K, K, kchunk), whole)


@pytest.mark.parametrize("M,N,K,kchunk", [(8, 8, 16384, 8192), (64, 96, 12000, 8192),
                                          (344, 600, 16000, 8192), (256, 256, 2560, 2048),
                                          (1336, 1592, 8200, 4128)])
def test_two_pieces(M, N, K, kchunk):
    A = random_bf16(M, K, seed=3).view(torch.int16)
    B = random_bf16(N, K, seed=4).view(torch.int16)
    first = product(A, B, kchunk, K, atomic=False)
    second = product(A[:, kchunk:], B[:, kchunk:], K - kchunk, K, atomic=False)
    for _ in range(3):
        assert torch.equal(product(A, B, K, K, kchunk), first + second)
