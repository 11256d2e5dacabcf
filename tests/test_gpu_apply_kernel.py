"""mf_apply_kernel names the kernel that an apply runs: with the built-in choice, a launch
shape, the deterministic assembly, spans past 32-bit offsets, and on general cells."""
import pytest

import workloads as W
from paper_2208_07129_amd import mfmv

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
    assert mfmv.lib().mf_apply_kernel(None, 4, 0) is None
