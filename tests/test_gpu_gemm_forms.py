"""The BF16 matrix product over its dispatch: the one-pass kernel for long batches at
the edges of its tiles, K ranges, layouts and epilogues, the tiled kernel with 128-row
tiles, its re-cut split of K, and operands whose offsets need 64 bits; against FP32
products of the BF16 operands (columns at the ends and in between), at the FP32
accumulation's 1e-6 of K max|A| max|B|."""
import numpy as np
import pytest

from paper_2208_07129_amd import mlp

from test_gpu_mlp import bf, dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
NAN16 = 0x7FC1


def random_bf16(*shape, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(*shape, device="cuda", generator=g).to(torch.bfloat16)


def columns_of(n):
    return np.unique(np.r_[0:40, n // 2 - 9:n // 2 + 9, n - 40:n])


def check(got, A, B, cols, post=lambda x: x, rel=0.0):
    """got (M x cols) against A B[:, cols]; rel: the rounding of a BF16 output."""
    Ah, Bh = A.float().cpu(), B[:, torch.as_tensor(cols, device=B.device)].float().cpu()
    ref = post((Ah @ Bh).numpy())
    tol = 1e-6 * float(Ah.abs().max() * Bh.abs().max()) * Ah.shape[1]
    assert np.all(np.abs(got - ref) <= tol + rel * np.abs(ref))


@pytest.mark.parametrize("M,N,K", [(8, 32768, 8), (24, 32776, 128), (344, 32896, 136),
                                   (40, 65544, 256), (344, 65792, 344), (16, 65528, 352),
                                   (344, 32840, 360), (56, 65600, 608), (24, 32800, 616),
                                   (136, 131080, 40)])
def test_long_batch(M, N, K):
    A = random_bf16(M, K + 8, seed=M + K)[:, :K]  # lda > K
    B = random_bf16(K, N, seed=N)
    bias = torch.linspace(-1, 1, M, device="cuda")
    cols = columns_of(N)
    idx = torch.as_tensor(cols, device="cuda")
    a16, b16 = A.view(torch.int16), B.view(torch.int16)
    f32 = torch.full((M, N), float("nan"), device="cuda")
    mlp.CellMLP._gemm(M, N, K, False, False, a16, K + 8, b16, N, out_f32=f32, ld_f32=N)
    check(f32[:, idx].cpu().numpy(), A, B, cols)
    assert not torch.isnan(f32).any()
    mlp.CellMLP._gemm(M, N, K, False, False, a16, K + 8, b16, N, bias=bias, out_f32=f32, ld_f32=N)
    hb = bias.cpu().numpy()[:, None]
    check(f32[:, idx].cpu().numpy(), A, B, cols, lambda x: x + hb)
    o16 = torch.full((M, N + 8), NAN16, dtype=torch.int16, device="cuda")  # ld > N
    mlp.CellMLP._gemm(M, N, K, False, False, a16, K + 8, b16, N, bias=bias, relu=True,
                      out_bf16=o16, ld_bf16=N + 8)
    got = o16.view(torch.bfloat16)
    check(got[:, idx].float().cpu().numpy(), A, B, cols, lambda x: np.maximum(x + hb, 0),
          rel=2.0 ** -8)
    assert not torch.isnan(got[:, :N].float()).any()
    assert torch.isnan(got[:, N:].float()).all()  # nothing past a row's end
    # A stored K x M, the mask of the backward pass
    At = A.t().contiguous()
    mask = random_bf16(M, N, seed=3)
    mlp.CellMLP._gemm(M, N, K, True, False, At.view(torch.int16), M, b16, N,
                      mask=mask.view(torch.int16), ldmask=N, out_bf16=o16, ld_bf16=N + 8)
    keep = (mask[:, idx].float() > 0).cpu().numpy()
    check(got[:, idx].float().cpu().numpy(), A, B, cols, lambda x: x * keep, rel=2.0 ** -8)


@pytest.mark.parametrize("kb", [8, 24, 128, 264])
@pytest.mark.parametrize("K", [32, 216, 512])
def test_long_batch_in_blocks(kb, K):
    M, blocks = 72, (33000 + kb - 1) // kb
    N = blocks * kb
    A, Bb = random_bf16(M, K, seed=K), random_bf16(blocks, K, kb, seed=kb)
    out = torch.full((blocks, M, kb), float("nan"), device="cuda")
    mlp.CellMLP._gemm(M, N, K, False, False, A.view(torch.int16), K, Bb.view(torch.int16), K * kb,
                      out_f32=out, ld_f32=M * kb, kb=kb)
    B = Bb.permute(1, 0, 2).reshape(K, N)
    cols = columns_of(N)
    got = out.permute(1, 0, 2).reshape(M, N)[:, torch.as_tensor(cols, device="cuda")]
    check(got.cpu().numpy(), A, B, cols)
    assert not torch.isnan(out).any()


@pytest.mark.parametrize("M,N,K,kchunk", [(344, 600, 8200, 4096), (8, 8, 40000, 8192),
                                          (136, 264, 20480, 32)])
def test_split_k(M, N, K, kchunk):
    """Weight gradients: pieces of K added atomically (FP32, any order)."""
    A, B = random_bf16(M, K, seed=1), random_bf16(N, K, seed=2)
    out = torch.zeros(M, N, device="cuda")
    mlp.CellMLP._gemm(M, N, K, False, True, A.view(torch.int16), K, B.view(torch.int16), K,
                      kchunk=kchunk, out_f32=out, ld_f32=N, atomic=True)
    check(out.cpu().numpy(), A, B.t(), np.arange(N))


@pytest.mark.parametrize("ta,tb", [(False, False), (True, False), (False, True), (True, True)])
def test_unaligned_outputs_and_large_tiles(ta, tb):
    """128-row tiles (4 x 130 of them) and outputs that only take single elements."""
    M, N, K = 392, 16520, 72
    A, B = random_bf16(M, K, seed=4), random_bf16(K, N, seed=5)
    As = (A.t() if ta else A).contiguous().view(torch.int16)
    Bs = (B.t() if tb else B).contiguous().view(torch.int16)
    buf = torch.zeros(M * (N + 1) + 1, device="cuda")
    out = buf[1:].view(M, N + 1)
    mlp.CellMLP._gemm(M, N, K, ta, tb, As, As.shape[1], Bs, Bs.shape[1], out_f32=out, ld_f32=N + 1)
    cols = columns_of(N)
    check(out[:, torch.as_tensor(cols, device="cuda")].cpu().numpy(), A, B, cols)
    assert float(buf[0]) == 0.0 and not out[:, N].any()


@pytest.mark.parametrize("ta,tb", [(False, False), (False, True)])
def test_offsets_beyond_32_bits(ta, tb):
    """A leading dimension so large that one step of K (or one tile of rows) spans
    more than 2 GiB."""
    M, K, N = 24, 40, 16
    big = (1 << 25) if not tb else (1 << 23)
    rows = K if not tb else N
    X = torch.zeros(rows * big, dtype=torch.int16, device="cuda").view(rows, big)
    A, B = random_bf16(M, K, seed=6), random_bf16(K, N, seed=7)
    Bs = B.t().contiguous() if tb else B
    X[:, :Bs.shape[1]] = Bs.view(torch.int16)
    out = torch.full((M, N), float("nan"), device="cuda")
    mlp.CellMLP._gemm(M, N, K, ta, tb, A.view(torch.int16), K, X, big, out_f32=out, ld_f32=N)
    check(out.cpu().numpy(), A, B, np.arange(N))
