"""The linear cell preconditioner with the gather inside the matrix product: the same bits
as the gather, the product and the assembly one after the other, over degrees, boundary
conditions, column counts that divide a workgroup's 128 and that do not, and the calls
that keep the separate form (few rows, odd leading dimension, many cells per workgroup)."""
import numpy as np
import pytest

import workloads as W
from paper_2208_07129_amd import mfmv, mlp

from test_gpu_mlp import small_op

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,n,k,ld,bc", [
    (2, (9, 8, 8), 64, 64, W.BC_PERIODIC), (2, (17, 16, 16), 8, 8, W.BC_DIRICHLET0),
    (3, (11, 10, 10), 40, 42, W.BC_NONE), (4, (8, 7, 7), 88, 88, W.BC_DIRICHLET0),
    (5, (7, 7, 7), 96, 99, W.BC_PERIODIC), (5, (7, 7, 7), 96, 100, W.BC_PERIODIC),
    (6, (5, 5, 6), 256, 256, W.BC_DIRICHLET0), (6, (13, 13, 13), 16, 16, W.BC_PERIODIC),
    (6, (9, 9, 9), 56, 56, W.BC_PERIODIC), (7, (5, 6, 5), 128, 128, W.BC_NONE),
    (4, (3, 2, 2), 128, 128, W.BC_PERIODIC)])
def test_same_bits_as_the_separate_steps(p, n, k, ld, bc):
    mesh, op = small_op(bc, p=p, n=n)
    diag = mfmv.diagonal(op)
    net = mlp.CellMLP(op, hidden=16, seed=2, out_scale=1.0, dscale=diag)
    F, Fp, H = net.F, net.Fp, net.H
    S = torch.randn(F, F, device="cuda")
    net.params[4][:F, H:H + F].copy_(0.1 * (S + S.t()))
    net.wbf[4].copy_(net.params[4].to(torch.bfloat16).view(torch.int16))
    R = torch.randn(op.ndofs, ld, dtype=torch.float64, device="cuda")[:, :k]
    Z, Z2 = torch.empty(2, op.ndofs, k, dtype=torch.float64, device="cuda")
    net.precondition(R, Z, diag, linear=True)
    b = net.gather(R, pou_sqrt=True, normalise=False, blocked=False)
    m = b["ld"]
    net._gemm(Fp, m, Fp, False, False, net.wbf[4][:, H:], H + Fp, b["X0"], m, out_f32=b["Y"], ld_f32=m)
    mfmv._check(mfmv.lib().mf_cell_scatter(
        op._h, k, b["Y"].data_ptr(), m, None, diag.data_ptr(), R.data_ptr(), ld, Z2.data_ptr(), k, 1,
        diag.data_ptr(), 0, None))
    torch.cuda.synchronize()
    assert torch.equal(Z, Z2)


def test_cell_linear_rejects_bad_arguments():
    _, op = small_op(W.BC_PERIODIC, p=2, n=(2, 2, 2))
    R = torch.zeros(op.ndofs, 16, dtype=torch.float64, device="cuda")
    S = torch.zeros(32, 32, dtype=torch.int16, device="cuda")
    X0 = torch.zeros(8 * 32 * 16, dtype=torch.int16, device="cuda")
    Y = torch.zeros(8 * 32 * 16, device="cuda")
    call = mfmv.lib().mf_cell_linear
    good = [op._h, 16, R.data_ptr(), 16, 32, S.data_ptr(), 32, X0.data_ptr(), Y.data_ptr(), 512, 1,
            None, None]
    assert call(*good) == 0
    for at, bad in ((1, 12), (3, 8), (4, 24), (6, 24), (9, 511), (2, None), (5, S.data_ptr() + 2)):
        args = list(good)
        args[at] = bad
        assert call(*args) == mfmv.MF_ERR_ARG, at
    torch.cuda.synchronize()
