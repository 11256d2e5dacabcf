"""The gather with two to eight cells per workgroup, which meshes of more than 512 cells (or
16 rows of a large cell) take: a last workgroup with fewer cells, columns that do not
divide its 64 lanes, and normalised inputs and targets, against the oracle."""
import numpy as np
import pytest

import workloads as W
from oracle import mlp_oracle as mo
from oracle.fe_oracle import constrained_mask
from paper_2208_07129_amd import mlp

from test_gpu_cell_rows import values
from test_gpu_mlp import dev, small_op

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 3, 7, 8, 21, 32])
@pytest.mark.parametrize("bc,n,p", [(W.BC_DIRICHLET0, (3, 11, 17), 2), (W.BC_PERIODIC, (5, 11, 23), 1),
                                    (W.BC_NONE, (7, 17, 37), 1), (W.BC_PERIODIC, (3, 2, 1), 6)])
def test_gather_over_many_cells(bc, n, p, k):
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
