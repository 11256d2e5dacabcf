"""mf_apply_kernel names the kernel that an apply runs: with the built-in choice, a launch
shape, the deterministic assembly, spans past 32-bit offsets, and on general cells."""
import numpy as np
import pytest

import workloads as W
from paper_2208_07129_amd import mfmv

from test_gpu_apply import build_pair, colrel, TOL

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

PAIR, BOX, PERS = "apply_pair_kernel", "apply_box_kernel", "apply_box_pers_kernel"


def cube(n, p, q=None, bc=W.BC_PERIODIC, lin=None):
    n = (n,) * 3 if isinstance(n, int) else n
    return mfmv.Operator(W.BoxMesh(n=n, bc=bc, lin=lin), p, q or p + 1, 0.5, None, 0.2)


def test_kernel_names():
    op = cube(4, 6)
    assert op.apply_kernel(64) == BOX                       # too few cells
    op.set_launch(False, 0)
    assert op.apply_kernel(64) == PAIR
    op.set_launch(False, 5)
    assert op.apply_kernel(64) == PERS
    op.set_launch(False, 10)
    assert op.apply_kernel(64) == "apply_mfma_kernel"
    op.set_launch(False, 0)
    op.set_deterministic(True)
    assert op.apply_kernel(64) == BOX
    op.set_deterministic(False)
    assert op.apply_kernel(64, "fp32") == "apply_vec32_kernel"
    assert op.apply_kernel(64, "bf16") == "apply_mixed_kernel"
    op.set_launch(True)
    assert op.apply_kernel(64) == "apply_f64_kernel"
    op = cube(2, 2)
    op.set_launch(False, 0)
    most = 0xF0000000 // (8 * op.ndofs)
    assert op.apply_kernel(most - 1) == PAIR and op.apply_kernel(most + 1) == BOX
    sheared = cube(2, 2, lin=((1.0, 0.2, 0.0), (0.0, 1.0, 0.0), (0.0, 0.0, 1.0)), bc=W.BC_NONE)
    assert sheared.apply_kernel(4) == "apply_f64_kernel"
    assert sheared.apply_kernel(4, "fp32") is None
    assert op.apply_kernel(0) is None
    assert mfmv.lib().mf_apply_kernel(None, 4, 0, 0) is None


def test_accumulating_apply():
    """More than three points per direction accumulate in the box kernel, whatever the
    storing form runs: by choice, by shape and after tuning."""
    for p, q, n, k in [(6, 7, 12, 64), (4, 5, 16, 64), (3, 4, 20, 32), (2, 4, 16, 33)]:
        op = cube(n, p, q)
        assert op.apply_kernel(k, accumulate=True) == BOX
        op.set_launch(False, 0)
        assert op.apply_kernel(k) == PAIR and op.apply_kernel(k, accumulate=True) == BOX
    for p, q, n, k in [(2, 3, 32, 1), (2, 3, 24, 64), (1, 3, 40, 16), (1, 2, 40, 4)]:
        assert cube(n, p, q).apply_kernel(k, accumulate=True) == PAIR
    op = cube((1, 30000, 1), 2)  # fewer cells in x than share a wavefront
    assert op.apply_kernel(1) == PAIR and op.apply_kernel(1, accumulate=True) == BOX
    op = cube(12, 4)
    op.set_launch(False, 0)
    op.tune(33)
    assert op.apply_kernel(33, accumulate=True) == BOX


@pytest.mark.parametrize("p,q,n,k", [(6, 7, (4, 5, 3), 33), (4, 5, (5, 4, 4), 64), (3, 4, (4, 6, 5), 17),
                                     (2, 4, (6, 5, 7), 9), (2, 3, (16, 17, 18), 33),
                                     (1, 3, (20, 20, 21), 20), (2, 3, (33, 16, 16), 1)])
def test_accumulating_apply_matches_the_oracle(p, q, n, k):
    mesh = W.BoxMesh(n=n, bc=W.BC_DIRICHLET0)
    op, orc = build_pair(mesh, p, q)
    rng = np.random.default_rng(p + k)
    X, Y0 = rng.uniform(-1, 1, (orc.ndofs, k)), rng.uniform(-1, 1, (orc.ndofs, k))
    ref = Y0 + orc.apply(X)
    ref[orc.constrained] = Y0[orc.constrained]
    for shape in (-1, 0):
        op.set_launch(False, shape)
        Y = torch.from_numpy(Y0).to("cuda")
        op.apply(torch.from_numpy(X).to("cuda"), Y, accumulate=True)
        assert colrel(Y.cpu().numpy(), ref) <= TOL


@pytest.mark.parametrize("p,q,n,pair,box", [
    # (columns of the register form, columns of the box kernel)
    (6, 7, 16, (9, 12, 32, 33, 64), (1, 2, 4, 8, 16, 24, 40)),
    (6, 7, 12, (33, 128), (1, 8, 40, 56, 64)),
    (4, 5, 24, (9, 16, 20, 24, 32, 64), (1, 2, 4, 8)),
    (3, 4, 20, (17, 20, 32, 40, 64), (1, 2, 8, 9, 16, 24)),
    (2, 3, 32, (1, 2, 4, 8, 16, 24, 64), ()),
    (2, 3, 8, (), (1, 2, 4, 8, 16, 24, 64)),
    (2, 4, 16, (33,), (1, 8, 16, 20, 24, 40, 64)),
    (1, 2, 40, (1, 4, 9, 16, 20, 32), (8, 24)),
    (1, 2, (7, 64, 64), (1, 4, 9, 12), (8, 16, 20, 24, 56, 64)),
    (1, 4, 40, (3, 4), (1, 8, 12, 16, 24, 64)),
    (5, 6, 20, (), (1, 9, 16, 64)),
    (8, 9, 12, (), (1, 8, 64)),
])
def test_choice_between_register_form_and_box_kernel(p, q, n, pair, box):
    """Narrow blocks, half-idle tiles and points per direction on both sides of the rule."""
    op = cube(n, p, q)
    for k in pair:
        assert op.apply_kernel(k) == PAIR, k
    for k in box:
        assert op.apply_kernel(k) in (BOX, PERS), k
