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


def plain_sweeps(A, sweeps):
    """The block method with numpy's rotations, one after the other: the path of signs that
    the kernel's rounds have to follow."""
    K = A.shape[0]
    A, V, nb = A.copy(), np.eye(K), K // 32
    pairs = lambda n, r: [sorted((0 if t == 0 else 1 + (t - 1 + r) % (n - 1),
                                  1 + (n - 2 - t + r) % (n - 1))) for t in range(n // 2)]
    for _ in range(sweeps):
        for r in range(nb - 1):
            J = np.zeros((K, K))
            for P, Q in pairs(nb, r):
                idx = np.r_[32 * P:32 * P + 32, 32 * Q:32 * Q + 32]
                B, W = A[np.ix_(idx, idx)].copy(), np.eye(64)
                for rr in range(63):
                    G = np.eye(64)
                    for p, q in pairs(64, rr):
                        if abs(B[p, q]) > 1e-300:
                            th = (B[q, q] - B[p, p]) / (2 * B[p, q])
                            t = (1.0 if th >= 0 else -1.0) / (abs(th) + np.sqrt(th * th + 1))
                            c = 1 / np.sqrt(t * t + 1)
                            G[p, p] = G[q, q] = c
                            G[p, q], G[q, p] = t * c, -t * c
                    B, W = G.T @ B @ G, W @ G
                J[np.ix_(idx, idx)] = W
            A, V = J.T @ A @ J, V @ J
    order = np.argsort(np.diag(A), kind="stable")
    return V[:, order]


@pytest.mark.parametrize("k", [128])
def test_signs_follow_the_plain_sweeps(k):
    """Well separated diagonal entries keep every rotation away from a tie, so the
    eigenvectors come out with the signs of the plain method."""
    rng = np.random.default_rng(5)
    Z = rng.standard_normal((k, k))
    A = np.diag(np.arange(k) * 1.0) + 0.02 * (Z + Z.T)
    _, V, st = mfmv.sym_eig(T(A))
    assert int(st.item()) == 0
    ref = plain_sweeps(A, 6)
    assert np.abs(V.cpu().numpy() - ref).max() <= 1e-9
