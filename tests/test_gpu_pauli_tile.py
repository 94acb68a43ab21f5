"""Pauli strings taken many to a sweep of the state (4 qubits and more) against
the oracle: x bits on run, tile and outer qubits, one string, more strings
than a sweep takes, strings with more x bits than a tile holds (grouped by x
instead), Y parts of every count, rows of a batch.

Tolerance: terms are FP64 products of at most 2^15 amplitudes of a normalised
state, summed in FP64, so 1e-12 absolute leaves two orders to spare."""

import numpy as np
import pytest

import oracle
from tests import pins

pytestmark = pytest.mark.gpu


def _strings(n, count, rng):
    out = [(0, 0), (1, 1), (1 << (n - 1), (1 << n) - 1), ((1 << n) - 1, (1 << n) - 1), (0, 1 << (n - 1))]
    for _ in range(count):
        x = z = 0
        for q in rng.permutation(n)[: int(rng.integers(1, n + 1 if rng.random() < 0.1 else 5))]:
            k = int(rng.integers(1, 4))
            x |= (k & 1) << int(q)
            z |= (k >> 1) << int(q)
        out.append((x, z))
    return out


@pytest.mark.parametrize("n, batch, count", [(3, 2, 9), (4, 2, 20), (5, 1, 40), (9, 3, 60), (10, 1, 0), (12, 2, 300),
                                             (13, 1, 30), (15, 2, 330)])
def test_matches_oracle(sv, n, batch, count):
    rng = np.random.default_rng(40 + n)
    strings = _strings(n, count, rng)
    rows = [pins.random_state(n, rng).astype(np.complex64) for _ in range(batch)]
    st = sv.State(n, batch)
    st.from_numpy(np.stack(rows))
    out = st.expval([(1.0, x, z) for x, z in strings])
    again = st.expval([(1.0, x, z) for x, z in strings])
    assert np.array_equal(out, again)
    for r in range(batch):
        ref = rows[r].astype(np.complex128)
        for t, (x, z) in enumerate(strings):
            assert abs(out[r, t] - oracle.expval_pauli(ref, n, x, z)[0]) < 1e-12, (r, t, x, z)
    # each string by itself (by x) takes the same value up to the order of the sums
    one = np.array([st.expval([(1.0, x, z)])[:, 0] for x, z in strings[:8]]).T
    assert np.max(np.abs(one - out[:, :8])) < 1e-12
