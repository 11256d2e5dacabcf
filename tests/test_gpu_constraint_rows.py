"""Hanging-node constraints over every degree (each number of masters per wavefront),
column counts at the edges of a tile: C reproduces constants, and its products
agree with those of C^T (the adjoint) to the rounding of the sums."""
import numpy as np
import pytest

import workloads as W
from paper_2208_07129_amd import mfmv

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", range(1, 11))
@pytest.mark.parametrize("nvec", [1, 63, 65])
def test_adjoint_and_constants(p, nvec):
    mesh = W.RefinedMesh(n=(3, 3, 3), lo=(0, 0, 0), hi=(1.0, 1.0, 1.0), bc=W.BC_NONE,
                         rlo=(1, 1, 1), rhi=(2, 2, 2))
    op = mfmv.RefinedOperator(mesh, p, p + 1, 0.5, None, 1.0)
    g = torch.Generator(device="cuda").manual_seed(p)
    X, Y = (torch.randn(2, op.ndofs, nvec + 2, dtype=torch.float64, device="cuda",
                        generator=g)[i][:, :nvec] for i in range(2))
    ones = op.distribute(torch.ones(op.ndofs, nvec, dtype=torch.float64, device="cuda"))
    assert float((ones - 1).abs().max()) <= 1e-12
    CX, CtY = X.clone(), Y.clone()
    op.distribute(CX)
    op.condense(CtY)
    torch.cuda.synchronize()
    a, b = (Y * CX).sum(0), (CtY * X).sum(0)
    scale = (Y.abs() * CX.abs()).sum(0)
    assert bool(((a - b).abs() <= 1e-12 * scale).all())
    slaves = torch.from_numpy(op.constrained_rows()).cuda()
    assert not bool(CtY[slaves].any())
