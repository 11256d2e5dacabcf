"""One to four columns: the assembly along memory rows of the box kernel's narrow tiles,
over every degree and quadrature, on meshes on both sides of its choice, against the CPU
oracle per column at 1e-12; accumulating, strided and deterministic forms."""
import numpy as np
import pytest

import workloads as W
from paper_2208_07129_amd import mfmv

from test_gpu_apply import build_pair, colrel, gpu_apply, TOL

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", range(1, 11))
@pytest.mark.parametrize("bc", [W.BC_PERIODIC, W.BC_DIRICHLET0, W.BC_NONE])
def test_narrow_every_degree(p, bc):
    n = (3, 2, 2) if p > 4 else (11, 10, 10)  # below and above 1024 cells
    mesh = W.BoxMesh(n=n, lo=(0.0, -0.5, 0.25), hi=(1.0, 1.0, 1.5), bc=bc)
    for q in range(p + 1, p + 4 if p <= 8 else p + 2):
        op, orc = build_pair(mesh, p, q)
        for nv in (1, 2, 3, 4) if q == p + 1 else (1, 3):
            X = np.random.default_rng(10 * p + nv).uniform(-1, 1, (orc.ndofs, nv))
            assert colrel(gpu_apply(op, X), orc.apply(X)) <= TOL, (p, q, bc, nv)


@pytest.mark.parametrize("p", [5, 6, 7, 8])
def test_narrow_large_meshes(p):
    """More than 1024 cells of a high degree: the same columns inside a wide block."""
    mesh = W.BoxMesh(n=(9, 11, 11), lo=(0, 0, 0), hi=(1.0, 0.8, 1.4), bc=W.BC_DIRICHLET0)
    Vq = np.sin(np.arange(9 * 11 * 11 * (p + 1) ** 3) * 0.37)
    op = mfmv.Operator(mesh, p, p + 1, 0.5, Vq, 0.1)
    X = torch.rand(op.ndofs, 8, dtype=torch.float64, device="cuda:0") - 0.5
    ref = op.apply(X)
    for nv in (1, 2, 3, 4):
        Y = torch.full((op.ndofs, nv + 3), 3.0, dtype=torch.float64, device="cuda:0")
        op.apply(X[:, :nv], Y[:, :nv])
        scale = float(ref.abs().max())
        assert float((Y[:, :nv] - ref[:, :nv]).abs().max()) <= 1e-12 * scale
        assert bool((Y[:, nv:] == 3.0).all())
        Z = Y[:, :nv].clone()
        op.apply(X[:, :nv], Z, accumulate=True)
        assert float((Z - 2 * ref[:, :nv]).abs().max()) <= 2e-12 * scale
    op.set_deterministic(True)
    Xc = X[:, :1].contiguous()
    assert torch.equal(op.apply(Xc), op.apply(Xc))
