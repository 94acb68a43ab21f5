"""Which backward the autograd layers take by default: matrix-core blocks or
tiles, as measured for training steps of each kind of circuit."""

import pytest

from paper_2511_19291_amd import circuits as C
from paper_2511_19291_amd import sv
from paper_2511_19291_amd.autograd import default_block_qubits

BLOCKS, TILES = sv.ADJOINT_MFMA, 0


def _bricks(n, layers, two, general):
    """Rotations with `general` of every 20 gates a U3, and bricks of CX or CRX."""
    b = C._Builder(n)
    for layer in range(layers):
        for q in range(n):
            if (q + layer * n) % 20 < general:
                b.gate("u3", [q], values=[0.1, 0.2, 0.3])
            else:
                b.gate(("rx", "ry", "rz")[q % 3], [q], values=[0.1])
        for q in range(layer % 2, n - 1, 2):
            b.gate("x" if two == "cx" else "rx", [q + 1], [q], values=[] if two == "cx" else [0.4])
    return b.build("bricks")


def _ladder(n, layers):
    """RY on every qubit, CRX down the line."""
    b = C._Builder(n)
    for _ in range(layers):
        for q in range(n):
            b.gate("ry", [q], values=[0.1])
        for q in range(n - 1):
            b.gate("rx", [q + 1], [q], values=[0.2])
    return b.build("ladder")


@pytest.mark.parametrize("circ, batch, want", [
    # controlled rotations in bricks (tiles : blocks, ms): 14.0 : 10.9, 14.9 : 11.2, 30.6 : 21.8; 24 qubits 7.4 : 6.7
    (_bricks(25, 8, "crx", 5), 1, BLOCKS), (_bricks(26, 4, "crx", 4), 1, BLOCKS), (_bricks(27, 4, "crx", 0), 1, BLOCKS),
    (_bricks(24, 8, "crx", 5), 1, BLOCKS),
    # in rows: 8.3 : 6.4, 14.4 : 10.5; 4.2 : 4.7 and 12.5 : 27.8 on fewer qubits
    (_bricks(21, 8, "crx", 5), 16, BLOCKS), (_bricks(25, 8, "crx", 5), 2, BLOCKS),
    (_bricks(20, 4, "crx", 2), 16, TILES), (_bricks(18, 4, "crx", 2), 256, TILES),
    # 3.7 : 4.5, 1.4 : 3.4 on fewer qubits
    (_bricks(23, 8, "crx", 3), 1, TILES), (_bricks(21, 8, "crx", 3), 1, TILES),
    # in ladders: 4.5 : 6.5, 9.0 : 10.9, 36.0 : 39.3
    (_ladder(24, 4), 1, TILES), (_ladder(25, 4), 1, TILES), (_ladder(27, 4), 1, TILES),
    # U3 among rotations: a quarter 23.6 : 21.7 on 27 qubits, a fifth 2.8 : 3.9 on 24
    (_bricks(27, 4, "cx", 5), 1, BLOCKS), (_bricks(24, 4, "cx", 4), 1, TILES),
    # rotations only; mostly U3
    (_bricks(27, 4, "cx", 0), 1, TILES), (C.rxry_ring(28, 10, 5), 1, TILES), (C.rxry_ring(25, 3, 5), 16, TILES),
    (_bricks(22, 4, "cx", 10), 1, BLOCKS), (_bricks(20, 4, "cx", 20), 1, TILES), (_bricks(27, 4, "cx", 20), 1, BLOCKS),
])
def test_backward_form(circ, batch, want):
    assert default_block_qubits(circ, batch) == want
