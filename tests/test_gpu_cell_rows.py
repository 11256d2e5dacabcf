"""The cell network's row kernels at the edges of their tilings, against the oracle or a
plain PyTorch reference: the gather with several cells per workgroup (column counts
that divide 64 and that do not, a last workgroup with fewer cells, the cell-blocked
layout), bias gradients and the loss gradient with and without aligned rows."""
import numpy as np
import pytest

import workloads as W
from oracle import mlp_oracle as mo
from oracle.fe_oracle import constrained_mask
from paper_2208_07129_amd import mfmv, mlp

from test_gpu_mlp import dev, small_op

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def values(t):
    return (t.cpu().numpy().view(np.uint16).astype(np.uint32) << 16).view(np.float32).astype(np.float64)


@pytest.mark.parametrize("k", [1, 2, 3, 7, 8, 16, 21, 32, 33, 64, 65])
@pytest.mark.parametrize("bc,n,p", [(W.BC_DIRICHLET0, (3, 3, 1), 2), (W.BC_PERIODIC, (5, 1, 2), 4),
                                    (W.BC_NONE, (1, 1, 1), 3)])
def test_gather_cells_per_workgroup(bc, n, p, k):
    mesh, op = small_op(bc, p=p, n=n)
    rng = np.random.default_rng(k + p)
    R, E = rng.uniform(-1, 1, (op.ndofs, k)), rng.uniform(-1, 1, (op.ndofs, k))
    R[constrained_mask(mesh, p)] = 0.0
    net = mlp.CellMLP(op, hidden=16, seed=1)
    b = net.gather(torch.from_numpy(R).to(dev()), torch.from_numpy(E).to(dev()))
    X, T, rho = mo.cell_inputs(mesh, p, R, E)
    rows, F = op.ncells * k, net.F
    np.testing.assert_allclose(b["rho"].cpu().numpy()[:rows], rho, rtol=1e-6)
    xs = values(b["X0"])
    assert np.all(np.abs(xs[:F, :rows].T - X) <= np.abs(X) * 2 ** -8 + 1e-30)
    assert not xs[F:, :rows].any() and not xs[:, rows:].any()
    np.testing.assert_allclose(b["T"].cpu().numpy()[:F, :rows].T, T, rtol=1e-6, atol=1e-12)
    if k % 8 == 0:  # cell-blocked, one block of Fp x k per cell
        flat = b["X0"][:, :rows].clone()
        Rd = torch.from_numpy(R).to(dev())
        net.gather(Rd, blocked=True)
        blk = b["X0"].reshape(-1)[:op.ncells * net.Fp * k].view(op.ncells, net.Fp, k)
        assert torch.equal(blk.permute(1, 0, 2).reshape(net.Fp, rows)[:F], flat[:F])


@pytest.mark.parametrize("M,N,pad,shift", [(3, 1, 7, 0), (8, 8191, 1, 0), (5, 40000, 8, 0),
                                           (4, 32768, 0, 0), (4, 33000, 0, 3)])
def test_row_sums(M, N, pad, shift):
    """FP32 sums of at most 40 terms a thread and 10 tree levels: 50 eps sum |x|."""
    buf = torch.randn(M * (N + pad) + shift, device="cuda").to(torch.bfloat16)
    X = buf[shift:].view(M, N + pad)
    out = torch.full((M,), 2.0, device="cuda")
    for acc in (0, 1):
        mfmv._check(mfmv.lib().mf_row_sums(M, N, X.data_ptr(), N + pad, out.data_ptr(), acc, None))
        torch.cuda.synchronize()
        ref = X[:, :N].double().sum(1) * (1 + acc)
        tol = 50 * 2.0 ** -23 * X[:, :N].double().abs().sum(1) * (1 + acc)
        assert bool(((out.double() - ref).abs() <= tol).all())


@pytest.mark.parametrize("F,Fp,N,ld,weights", [(5, 8, 1, 8, True), (8, 8, 1029, 1032, False),
                                               (27, 32, 4096, 4096, True), (27, 32, 2050, 2051, True)])
def test_mse_grad(F, Fp, N, ld, weights):
    Y, T = torch.randn(Fp, ld, device="cuda"), torch.randn(Fp, ld, device="cuda")
    w = torch.rand(N, device="cuda") if weights else None
    dY = torch.full((Fp, ld), 7, dtype=torch.int16, device="cuda")
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    scale = 0.25
    mfmv._check(mfmv.lib().mf_mse_grad(F, Fp, N, Y.data_ptr(), T.data_ptr(), ld,
                                       None if w is None else w.data_ptr(), scale, dY.data_ptr(),
                                       loss.data_ptr(), None))
    torch.cuda.synchronize()
    d = (Y - T)[:F, :N]
    wr = torch.ones(N, device="cuda") if w is None else w
    ref = float((scale * wr.double() * d.double() ** 2).sum())
    assert abs(float(loss.item()) - ref) <= 1e-10 * ref
    got = dY.view(torch.bfloat16).float()
    want = 2 * scale * wr * d
    assert bool(((got[:F, :N] - want).abs() <= 2.0 ** -8 * want.abs()).all())
    assert not got[F:, :N].any() and bool((dY[:, N:] == 7).all())


@pytest.mark.parametrize("F,N,nrows,K,weights", [(343, 32768, 32761, 600, True),
                                                 (27, 65536, 65536, 96, True),
                                                 (125, 33000, 32993, 256, False),
                                                 (216, 40000, 40000, 352, True),
                                                 (64, 1032, 1030, 64, True)])
def test_last_layer_with_its_loss_gradient(F, N, nrows, K, weights):
    """The bits of the product followed by the loss gradient (long batches form it in the
    product's epilogue); the loss up to the order of its double sums."""
    Fp = (F + 7) // 8 * 8
    A = torch.randn(Fp, K, device="cuda").to(torch.bfloat16).view(torch.int16)
    B = torch.randn(K, N, device="cuda").to(torch.bfloat16).view(torch.int16)
    bias, T = torch.randn(Fp, device="cuda"), torch.randn(Fp, N, device="cuda")
    w = torch.rand(N, device="cuda") if weights else None
    wp, s, lib = None if w is None else w.data_ptr(), 0.125, mfmv.lib()
    loss = torch.zeros(2, dtype=torch.float64, device="cuda")
    Y, Yw = torch.zeros(2, Fp, N, device="cuda")
    d0, d1 = torch.zeros(2, Fp, N, dtype=torch.int16, device="cuda")
    mlp.CellMLP._gemm(Fp, N, K, False, False, A, K, B, N, bias=bias, out_f32=Y, ld_f32=N)
    mfmv._check(lib.mf_mse_grad(F, Fp, nrows, Y.data_ptr(), T.data_ptr(), N, wp, s, d0.data_ptr(),
                                loss[:1].data_ptr(), None))
    mfmv._check(lib.mf_mlp_loss_grad(F, Fp, N, nrows, K, A.data_ptr(), K, B.data_ptr(),
                                     bias.data_ptr(), T.data_ptr(), N, wp, s, d1.data_ptr(),
                                     Yw.data_ptr(), loss[1:].data_ptr(), None))
    torch.cuda.synchronize()
    assert torch.equal(d0, d1)
    a, b = loss.tolist()
    assert abs(a - b) <= 1e-12 * a
