"""The block-Jacobi eigen-solver where its rotations are special: equal diagonal entries
(angles of pi/4 in every first round), scales far from one, and blocks that no sweep
can diagonalise."""
import numpy as np
import pytest

from paper_2208_07129_amd import mfmv

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("k", [65, 127, 129, 256])
@pytest.mark.parametrize("scale", [2.0 ** -400, 1.0, 2.0 ** 400])
def test_constant_diagonal_and_scale(k, scale):
    """A Toeplitz block (all diagonal entries equal); each eigenvalue is within
    4 k eps ||A|| of LAPACK's, as for two backward stable methods."""
    i = np.arange(k)
    A = scale / (1.0 + np.abs(i[:, None] - i[None, :]))
    w, V, st = mfmv.sym_eig(T(A))
    assert int(st.item()) == 0
    wh, Vh = w.cpu().numpy() / scale, V.cpu().numpy()
    ref = np.linalg.eigvalsh(A / scale)
    tol = 4 * k * np.finfo(np.float64).eps
    np.testing.assert_allclose(wh, ref, rtol=0, atol=tol * np.abs(ref).max())
    assert np.abs(A / scale @ Vh - Vh * wh).max() <= 10 * tol * np.abs(ref).max()
    assert np.abs(Vh.T @ Vh - np.eye(k)).max() <= tol


@pytest.mark.parametrize("k", [70, 192])
def test_not_a_number_is_reported(k):
    A = np.eye(k)
    A[3, 5] = A[5, 3] = np.nan
    _, _, st = mfmv.sym_eig(T(A))
    assert int(st.item()) == 1
