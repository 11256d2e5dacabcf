"""GPU parity of the Chebyshev step in the register-resident form (launch shape 0,
q <= 7) against the CPU oracle, per column at 1e-12 relative error: every degree, the
boundary conditions, one-cell periodic directions, segments of several cells with a
ragged last one, partial column tiles, strided rows, the three uses of Xp."""
import numpy as np
import pytest

import workloads as W
from paper_2208_07129_amd import mfmv

from test_gpu_cheb import T, colrel, dev, fo, vfun

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

PQ = [(p, q) for p in range(1, 7) for q in range(p + 1, min(p + 3, 7) + 1)]


def check(p, q, n, bc, nvecs, pad=0):
    mesh = W.BoxMesh(n=n, lo=(0.0, -0.5, 0.25), hi=(1.0, 1.0, 1.5), bc=bc)
    op = mfmv.Operator(mesh, p, q, 0.5, vfun(mfmv.quad_points(mesh, q)), 0.2)
    op.set_launch(False, 0)
    orc = fo.Oracle(mesh, p, q, 0.5, vfun, 0.2)
    m = orc.lumped_mass()
    D_ref = np.zeros_like(m)
    D_ref[~orc.constrained] = 1.0 / np.sqrt(m[~orc.constrained])
    D = D_ref.copy()
    D[orc.constrained] = np.nan  # never read into a result
    rng = np.random.default_rng(100 * p + q)
    a, b, c = 1.7, -0.6, 0.35
    for nv in nvecs:
        Y, Xp = rng.uniform(-1, 1, (2, orc.ndofs, nv))
        wide = lambda v: torch.cat([T(v), torch.full((orc.ndofs, pad), 7.0, dtype=torch.float64,
                                                     device=dev())], 1)[:, :nv]
        for mode in ("none", "separate", "inplace"):
            Yd = wide(Y)
            Out = wide(Xp if mode == "inplace" else np.full_like(Xp, np.nan))
            Xd = None if mode == "none" else (Out if mode == "inplace" else wide(Xp))
            mfmv.cheb_step(op, T(D), Yd, Xd, Out, a, b, c)
            torch.cuda.synchronize()
            ref = orc.cheb_step(D_ref, Y, None if mode == "none" else Xp, a, b, c)
            got = Out.cpu().numpy()
            assert colrel(got, ref) <= 1e-12, (p, q, n, bc, nv, mode)
            assert np.all(got[orc.constrained] == 0.0)


@pytest.mark.parametrize("p,q", PQ)
@pytest.mark.parametrize("bc", [W.BC_PERIODIC, W.BC_DIRICHLET0, W.BC_NONE])
def test_every_degree(p, q, bc):
    check(p, q, (3, 5, 2), bc, (16, 19))


@pytest.mark.parametrize("n", [(1, 1, 1), (1, 1, 3), (2, 1, 1), (1, 4, 1), (2, 7, 2)])
@pytest.mark.parametrize("bc", [W.BC_PERIODIC, W.BC_NONE])
def test_short_directions(n, bc):
    for p in (2, 3, 6):
        check(p, p + 1, n, bc, (1, 5, 33))


def test_strided_rows():
    check(4, 5, (3, 2, 2), W.BC_DIRICHLET0, (3, 17), pad=6)


def test_built_in_choice_on_a_long_mesh():
    """Segments of several cells (the built-in choice takes this form here)."""
    mesh = W.BoxMesh(n=(20, 21, 20), lo=(0, 0, 0), hi=(1.0, 1.0, 1.0), bc=W.BC_DIRICHLET0)
    op = mfmv.Operator(mesh, 2, 3, 0.5, vfun(mfmv.quad_points(mesh, 3)), 0.2)
    D = mfmv.gll_mass(op, inv_sqrt=True)
    Y, Xp = torch.rand(2, op.ndofs, 32, dtype=torch.float64, device=dev())
    outs = []
    for cfg in (-1, 0, 1):
        op.set_launch(False, cfg)
        outs.append(torch.empty_like(Y))
        mfmv.cheb_step(op, D, Y, Xp, outs[-1], 1.3, 0.4, -0.2)
    torch.cuda.synchronize()
    scale = float(outs[2].abs().max())
    for o in outs[:2]:
        assert float((o - outs[2]).abs().max()) <= 1e-13 * scale
