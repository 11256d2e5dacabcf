"""Cached FP64 tuning: an entry belongs to one set of launch shapes and one mesh shape.  An
entry under the former key (no set, no extents), whose shape 0 was another kernel, is not
taken, and meshes of equal cell count keep an entry each."""
import json

import pytest

import workloads as W
from paper_2208_07129_amd import mfmv

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def op_of(n):
    return mfmv.Operator(W.BoxMesh(n=n, bc=W.BC_PERIODIC), 2, 3, 0.5, None, 0.2)


def test_entry_of_the_former_shapes_is_not_taken(tmp_path):
    cache, op = tmp_path / "t.json", op_of((4, 4, 4))
    op.tune(8, "fp64", str(cache))
    (key, val), = json.load(open(cache)).items()
    former = key.split("/")[0] + "/p2q3/cells64/nvec8/fp64"
    assert key != former and key.endswith("/p2q3/cells64/nvec8/fp64")
    cache.write_text(json.dumps({former: {"cfg": 0, "ms": []}}))
    rec = op_of((4, 4, 4)).tune(8, "fp64", str(cache))
    assert rec["ms"]                                        # timed, not taken from the file
    assert set(json.load(open(cache))) == {former, key}     # and the other entry is left alone


def test_meshes_of_equal_cell_count(tmp_path):
    cache = str(tmp_path / "t.json")
    for n in [(4, 4, 4), (64, 1, 1), (1, 64, 1)]:
        assert op_of(n).tune(8, "fp64", cache)["ms"]
        assert not op_of(n).tune(8, "fp64", cache)["ms"]    # the second time from the file
    assert len(json.load(open(cache))) == 3


def test_mixed_keys_are_as_before(tmp_path):
    cache = tmp_path / "t.json"
    op_of((4, 4, 4)).tune(8, "fp32", str(cache))
    (key, _), = json.load(open(cache)).items()
    assert key.count("/") == 4 and key.split("/")[1] == "p2q3"
