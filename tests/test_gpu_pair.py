"""GPU parity of the register-resident FP64 apply (launch shape 0, q <= 7: one
wavefront per line of cells, matrix-core z contractions) against the CPU oracle,
per column at 1e-12 relative error: every degree and quadrature it is built for, the
column counts at the edges of its tiles (1, 2, 4, 8, 16 columns per wavefront),
boundary conditions, one-cell periodic directions, segments of several cells with a
ragged last one, the accumulating form, strided multivectors, and the box kernel where
its offsets do not reach."""
import numpy as np
import pytest

import workloads as W
from paper_2208_07129_amd import mfmv

from test_gpu_apply import build_pair, colrel, gpu_apply, TOL

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

PQ = [(p, q) for p in range(1, 7) for q in range(p + 1, min(p + 3, 7) + 1)]


@pytest.mark.parametrize("p,q", PQ)
@pytest.mark.parametrize("bc", [W.BC_PERIODIC, W.BC_DIRICHLET0, W.BC_NONE])
def test_pair_every_degree(p, q, bc):
    mesh = W.BoxMesh(n=(5, 3, 2), lo=(0.0, -0.5, 0.25), hi=(1.0, 1.0, 1.5), bc=bc)
    op, orc = build_pair(mesh, p, q)
    op.set_launch(False, 0)
    for nv in (1, 2, 3, 5, 8, 9, 16, 17, 33):
        X = np.random.default_rng(100 * p + nv + bc).uniform(-1, 1, (orc.ndofs, nv))
        assert colrel(gpu_apply(op, X), orc.apply(X)) <= TOL, (p, q, bc, nv)


@pytest.mark.parametrize("n", [(1, 1, 1), (1, 1, 3), (2, 1, 1), (1, 4, 1)])
def test_pair_one_cell_periodic(n):
    mesh = W.BoxMesh(n=n, lo=(0, 0, 0), hi=(1.0, 0.8, 1.4), bc=W.BC_PERIODIC)
    for p in (2, 4, 6):
        op, orc = build_pair(mesh, p, p + 1)
        op.set_launch(False, 0)
        for nv in (1, 6, 20):
            X = np.random.default_rng(p + nv).uniform(-1, 1, (orc.ndofs, nv))
            assert colrel(gpu_apply(op, X), orc.apply(X)) <= TOL, (n, p, nv)


@pytest.mark.parametrize("bc", [W.BC_PERIODIC, W.BC_DIRICHLET0, W.BC_NONE])
def test_pair_segments(bc):
    """33 x 7 x 32 cells, 65 columns: segments of four and three cells along y."""
    mesh = W.BoxMesh(n=(33, 7, 32), lo=(0, 0, 0), hi=(3.0, 1.0, 2.0), bc=bc)
    op, orc = build_pair(mesh, 2, 3)
    X = np.random.default_rng(5 + bc).uniform(-1, 1, (orc.ndofs, 65))
    ref = orc.apply(X)
    for cfg in (0, -1):
        op.set_launch(False, cfg)
        assert colrel(gpu_apply(op, X), ref) <= TOL, (bc, cfg)


def test_pair_accumulate_and_strides():
    mesh = W.BoxMesh(n=(3, 4, 2), lo=(0, 0, 0), hi=(1.5, 1.0, 1.0), bc=W.BC_DIRICHLET0)
    op, orc = build_pair(mesh, 6, 7)
    op.set_launch(False, 0)
    rng = np.random.default_rng(3)
    for nv in (1, 7, 21):
        X, Y0 = rng.uniform(-1, 1, (orc.ndofs, nv)), rng.uniform(-1, 1, (orc.ndofs, nv))
        ref = Y0 + orc.apply(X)
        ref[orc.constrained] = Y0[orc.constrained]   # constrained rows are left unchanged
        Xd = torch.full((orc.ndofs, nv + 3), np.nan, dtype=torch.float64, device="cuda")
        Yd = torch.full((orc.ndofs, nv + 6), 7.0, dtype=torch.float64, device="cuda")
        Xd[:, 2:nv + 2] = torch.from_numpy(X)
        Yd[:, 5:nv + 5] = torch.from_numpy(Y0)
        op.apply(Xd[:, 2:nv + 2], Yd[:, 5:nv + 5], accumulate=True)
        got = Yd.cpu().numpy()
        assert colrel(got[:, 5:nv + 5], ref) <= TOL, nv
        assert (got[:, :5] == 7.0).all() and (got[:, nv + 5:] == 7.0).all()
        op.apply(Xd[:, 2:nv + 2], Yd[:, 5:nv + 5])
        assert colrel(Yd.cpu().numpy()[:, 5:nv + 5], orc.apply(X)) <= TOL, nv


def test_pair_constrained_rows_ignored():
    """NaN and infinity in constrained rows of X do not enter the product."""
    mesh = W.BoxMesh(n=(2, 2, 3), lo=(0, 0, 0), hi=(1, 1, 1), bc=W.BC_DIRICHLET0)
    op, orc = build_pair(mesh, 4, 5)
    op.set_launch(False, 0)
    X = np.random.default_rng(9).uniform(-1, 1, (orc.ndofs, 10))
    ref = orc.apply(X)
    X[orc.constrained, ::2] = np.nan
    X[orc.constrained, 1::2] = np.inf
    got = gpu_apply(op, X)
    assert colrel(got, ref) <= TOL and (got[orc.constrained] == 0).all()


def test_pair_long_span_takes_box_kernel():
    """A leading dimension that takes the span past the 32-bit offsets."""
    mesh = W.BoxMesh(n=(2, 3, 2), lo=(0, 0, 0), hi=(1, 1, 1), bc=W.BC_NONE)
    op, orc = build_pair(mesh, 2, 3)
    op.set_launch(False, 0)
    ld = 0x100000000 // (8 * orc.ndofs) + 1
    X = np.random.default_rng(11).uniform(-1, 1, (orc.ndofs, 4))
    Xd = torch.zeros(orc.ndofs * ld, dtype=torch.float64, device="cuda").view(orc.ndofs, ld)
    Xd[:, :4] = torch.from_numpy(X)
    Y = op.apply(Xd[:, :4], torch.empty(orc.ndofs, 4, dtype=torch.float64, device="cuda"))
    assert colrel(Y.cpu().numpy(), orc.apply(X)) <= TOL
