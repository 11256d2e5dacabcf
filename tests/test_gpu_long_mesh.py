"""A mesh of very many cells along y: the register-resident form's work split is made on
every call, so it may not look at every length of a segment."""
import time

import pytest

import workloads as W
from paper_2208_07129_amd import mfmv

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_enqueueing_on_a_long_mesh():
    op = mfmv.Operator(W.BoxMesh(n=(1, 1 << 20, 1), bc=W.BC_PERIODIC), 1, 2, 0.5, None, 0.2)
    op.set_launch(False, 0)
    X = torch.rand(op.ndofs, 2, dtype=torch.float64, device="cuda")
    Y = torch.empty_like(X)
    op.apply(X, Y)
    torch.cuda.synchronize()
    t = time.perf_counter()
    for _ in range(10):
        op.apply(X, Y)
    t = (time.perf_counter() - t) / 10
    torch.cuda.synchronize()
    assert t < 1e-3   # some 2000 lengths; 2^20 of them take over 10 ms
    op.set_launch(False, 9)   # a box kernel shape
    ref = op.apply(X)
    assert float((Y - ref).norm() / ref.norm()) < 1e-13
