"""mf_mlp_loss_grad writes every column of dYt: zeros from nrows to N whichever path forms the
gradient (in the product's epilogue on long batches, by the loss kernel on short ones, on a
long K range and where rows start on 4 bytes only)."""
import pytest

from paper_2208_07129_amd import mfmv, mlp

from test_gpu_gemm_forms import random_bf16

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F,N,nrows,K,shift", [(27, 32, 1, 32, 0), (64, 1032, 1030, 64, 0),
                                               (30, 2048, 1025, 96, 0), (27, 1032, 1029, 40, 1),
                                               (27, 32768, 32761, 616, 0), (27, 32768, 32761, 96, 0),
                                               (125, 33000, 20001, 256, 0)])
def test_columns_past_the_rows(F, N, nrows, K, shift):
    Fp = (F + 7) // 8 * 8
    A, B = random_bf16(Fp, K, seed=1), random_bf16(K, N, seed=2)
    bias, w = torch.randn(Fp, device="cuda"), torch.rand(nrows, device="cuda")
    T = torch.randn(Fp * N + shift, device="cuda")[shift:].view(Fp, N)
    Y = torch.empty(Fp, N, device="cuda")
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    d = torch.full((Fp, N), 0x3F80, dtype=torch.int16, device="cuda")
    mfmv._check(mfmv.lib().mf_mlp_loss_grad(F, Fp, N, nrows, K, A.data_ptr(), K, B.data_ptr(),
                                            bias.data_ptr(), T.data_ptr(), N, w.data_ptr(), 0.125,
                                            d.data_ptr(), Y.data_ptr(), loss.data_ptr(), None))
    torch.cuda.synchronize()
    got = d.view(torch.bfloat16).float()
    assert not got[:, nrows:].any() and not got[F:].any()
    y = A.float().cpu() @ B.float()[:, :nrows].cpu() + bias.cpu()[:, None]
    want = 0.25 * w.cpu() * (y - T[:, :nrows].cpu())[:F]
    err = (got[:F, :nrows].cpu() - want).abs()
    # the gradient's BF16 rounding and the FP32 product's 1e-6 of K max|A| max|B|
    tol = 0.25 * 1e-6 * K * float(A.float().abs().max() * B.float().abs().max())
    assert bool((err <= 2.0 ** -8 * want.abs() + tol).all())


@pytest.mark.parametrize("Fp,N,K", [(8, 32760, 64), (8, 32768, 64), (24, 32768, 608), (24, 32768, 616),
                                    (4096, 32768, 8), (4104, 32768, 8)])
@pytest.mark.parametrize("shift", [0, 1, 2])
def test_both_sides_of_the_fused_form(Fp, N, K, shift):
    """At each limit of the product with a loss epilogue, the bits of the product followed by
    the loss gradient: no call may fall through to a product without its targets.  shift:
    targets (and, at 2, the gradient) that start off their alignment."""
    F, nrows, s, lib = Fp - 3, N - 5, 0.5, mfmv.lib()
    A, B = random_bf16(Fp, K, seed=5).view(torch.int16), random_bf16(K, N, seed=6).view(torch.int16)
    bias = torch.randn(Fp, device="cuda")
    T = torch.randn(Fp * N + shift, device="cuda")[shift:].view(Fp, N)
    g = torch.zeros(2, Fp * N + shift, dtype=torch.int16, device="cuda")
    d0, d1 = (x[shift if shift > 1 else 0:][:Fp * N].view(Fp, N) for x in g)
    loss = torch.zeros(2, dtype=torch.float64, device="cuda")
    Y = torch.empty(Fp, N, device="cuda")
    mlp.CellMLP._gemm(Fp, N, K, False, False, A, K, B, N, bias=bias, out_f32=Y, ld_f32=N)
    mfmv._check(lib.mf_mse_grad(F, Fp, nrows, Y.data_ptr(), T.data_ptr(), N, None, s, d0.data_ptr(),
                                loss[:1].data_ptr(), None))
    mfmv._check(lib.mf_mlp_loss_grad(F, Fp, N, nrows, K, A.data_ptr(), K, B.data_ptr(),
                                     bias.data_ptr(), T.data_ptr(), N, None, s, d1.data_ptr(),
                                     Y.data_ptr(), loss[1:].data_ptr(), None))
    torch.cuda.synchronize()
    assert torch.equal(d0, d1)
    a, b = loss.tolist()
    assert a > 0 and abs(a - b) <= 1e-12 * a
