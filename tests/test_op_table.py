"""OpTable's packed words against the sv_op fields they stand for."""

import numpy as np
import pytest

from paper_2511_19291_amd import circuits as C
from paper_2511_19291_amd import sv


@pytest.mark.parametrize("seed", range(4))
def test_fields(seed):
    circ = C.random_circuit(9, 80, seed, max_controls=3)
    ops = list(circ.ops) + [C.Op("matrix", (2, 5), (1,)), C.Op("u3", (0,), (), (4, 5, 6)), C.Op("rx", (np.int64(3),), (), (2**32 + 1,))]
    mats = {len(circ.ops): np.arange(16).reshape(4, 4) + 1j}
    for chosen in (ops, ops[:-1], ops[:1], []):
        t = sv.OpTable(chosen, mats)
        assert t.n == len(chosen)
        for o, op in zip(t.arr, chosen):
            assert (o.kind, o.n_targets, o.n_controls) == (sv.KINDS[op.kind], len(op.targets), len(op.controls))
            assert list(o.targets) == list(op.targets) + [0] * (2 - len(op.targets))
            assert list(o.controls) == list(op.controls) + [0] * (3 - len(op.controls))
            assert list(o.param) == ([p % 2**32 for p in op.params] + [-1] * 3)[:3]
            assert bool(o.matrix) == (op.kind == "matrix")
        if len(chosen) > len(circ.ops):
            assert t.arr[len(circ.ops)].matrix[3] == 1.0 and t.arr[len(circ.ops)].matrix[2] == 1.0


def test_refused():
    with pytest.raises(KeyError):
        sv.OpTable([C.Op("nope", (0,))])
    with pytest.raises(IndexError):
        sv.OpTable([C.Op("x", (0,), (1, 2, 3, 4))])
    with pytest.raises(TypeError):
        sv.OpTable([C.Op("x", (1.5,))])
    with pytest.raises(TypeError):
        sv.OpTable([C.Op("matrix", (0,))])
