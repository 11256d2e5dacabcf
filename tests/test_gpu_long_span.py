"""Register-resident apply and Chebyshev step on multivectors that span 2 to 3.75 GiB, where
sizes and offsets no longer fit a signed 32-bit number, and just past the limit, where
the box kernel runs: against the CPU oracle, with zero-Dirichlet rows (dropped
accesses), separate row strides of X and Y, and NaN between the columns of two rows."""
import numpy as np
import pytest

import workloads as W
from oracle import fe_oracle as fo
from paper_2208_07129_amd import mfmv

from test_gpu_apply import build_pair, colrel, TOL
from test_gpu_cheb import T, vfun

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GIB = 1 << 30
LIMIT = 0xF0000000  # bytes


def spread(V, span, fill=float("nan")):
    """The columns of V at the start of rows whose stride makes the span just `span` bytes at
    most (or the first stride past it for a negative span)."""
    n, k = V.shape
    ld = (abs(span) // 8 - k) // (n - 1) + (span < 0)
    assert ld > k and (((n - 1) * ld + k) * 8 < LIMIT) == (span > 0)
    buf = torch.full((n * ld,), fill, dtype=torch.float64, device="cuda").view(n, ld)
    buf[:, :k] = torch.from_numpy(V)
    return buf


@pytest.mark.parametrize("p,q,k", [(2, 3, 5), (6, 7, 17), (4, 5, 16), (1, 2, 1)])
@pytest.mark.parametrize("bc", [W.BC_DIRICHLET0, W.BC_PERIODIC])
@pytest.mark.parametrize("xspan,yspan", [(int(3.5 * GIB), int(2.2 * GIB)),
                                         (int(2.2 * GIB), LIMIT - 8), (-LIMIT, int(2.2 * GIB)),
                                         (int(2.2 * GIB), -LIMIT)])
def test_apply(p, q, k, bc, xspan, yspan):
    op, orc = build_pair(W.BoxMesh(n=(2, 3, 2), lo=(0, 0, 0), hi=(1, 1.5, 1), bc=bc), p, q)
    op.set_launch(False, 0)
    X = np.random.default_rng(p + k).uniform(-1, 1, (orc.ndofs, k))
    X[orc.constrained] = 0.0
    Xd, Yd = spread(X, xspan), spread(np.full_like(X, 5.0), yspan, fill=7.0)
    op.apply(Xd[:, :k], Yd[:, :k])
    got, ref = Yd[:, :k].cpu().numpy(), orc.apply(X)
    assert colrel(got, ref) <= TOL
    assert np.abs(got[-3:] - ref[-3:]).max() <= TOL * np.abs(ref).max()
    assert bool((Yd[:, k] == 7.0).all()) and bool((Yd[:, -1] == 7.0).all())


@pytest.mark.parametrize("p,q,k", [(2, 3, 17), (6, 7, 16)])
@pytest.mark.parametrize("bc", [W.BC_DIRICHLET0, W.BC_NONE])
@pytest.mark.parametrize("span", [int(3.5 * GIB), LIMIT - 8, -LIMIT])
@pytest.mark.parametrize("mode", ["none", "separate", "inplace"])
def test_cheb_step(p, q, k, bc, span, mode):
    mesh = W.BoxMesh(n=(2, 3, 2), lo=(0.0, -0.5, 0.25), hi=(1.0, 1.0, 1.5), bc=bc)
    op = mfmv.Operator(mesh, p, q, 0.5, vfun(mfmv.quad_points(mesh, q)), 0.2)
    op.set_launch(False, 0)
    orc = fo.Oracle(mesh, p, q, 0.5, vfun, 0.2)
    D = np.zeros(orc.ndofs)
    D[~orc.constrained] = 1.0 / np.sqrt(orc.lumped_mass()[~orc.constrained])
    Y, Xp = np.random.default_rng(p).uniform(-1, 1, (2, orc.ndofs, k))
    a, b, c = 1.7, -0.6, 0.35
    Yd = spread(Y, span)
    Out = spread(Xp if mode == "inplace" else np.full_like(Xp, np.nan), span, fill=7.0)
    Xd = None if mode == "none" else Out if mode == "inplace" else spread(Xp, span)
    mfmv.cheb_step(op, T(D), Yd[:, :k], None if Xd is None else Xd[:, :k], Out[:, :k], a, b, c)
    torch.cuda.synchronize()
    ref = orc.cheb_step(D, Y, None if mode == "none" else Xp, a, b, c)
    got = Out[:, :k].cpu().numpy()
    assert colrel(got, ref) <= 1e-12 and np.all(got[orc.constrained] == 0.0)
    assert np.abs(got[-3:] - ref[-3:]).max() <= 1e-12 * np.abs(ref).max()
    assert bool((Out[:, k] == 7.0).all()) and bool((Out[:, -1] == 7.0).all())
