"""Several fused blocks per sweep (13 qubits and more) against the same blocks
applied one call at a time, the sweep of its own that every single block keeps:
blocks of 1..5 qubits in any target order on low, high and mixed qubits, more
blocks on one tile than a launch takes, six-qubit blocks among the others, rows
with matrices of their own, states of one tile and of several.

BF16x3 blocks keep their order and arithmetic: equal to the bit. FP32 blocks on
different qubits may change places: each block rounds at 64 products of 2^-24,
about 1e-6 of the state's norm at worst, so 1e-7 per block in norm leaves room
where roundings add up at random."""

import numpy as np
import pytest

from tests import pins

pytestmark = pytest.mark.gpu


def _blocks(n, count, rng, widths=(1, 2, 3, 4, 5), qubits=None, rows=0):
    out = []
    for _ in range(count):
        k = int(rng.choice(widths))
        pool = np.arange(6, n) if k == 6 else (np.arange(n) if qubits is None else np.asarray(qubits))
        t = [int(q) for q in rng.permutation(pool)[:k]]
        u = [pins.haar_unitary(1 << k, rng) for _ in range(max(rows, 1))]
        out.append((t, np.stack(u) if rows else u[0]))
    return out


def _run(sv, n, batch, psi, calls, mode, rows):
    st = sv.State(n, batch)
    st.from_numpy(psi)
    for c in calls:
        (st.apply_fused_rows if rows else st.apply_fused)(c, mode)
    return st.to_numpy()


@pytest.mark.parametrize("n, batch, count, widths, low, rows", [
    (13, 1, 12, (1, 2, 3, 4, 5), False, False), (13, 2, 150, (1, 2), True, False), (14, 3, 20, (5,), False, False),
    (15, 1, 30, (2, 3, 5, 6), False, False), (17, 2, 30, (4, 5), False, True), (20, 1, 40, (1, 3, 5), False, False),
    (22, 1, 25, (5,), False, False)])
@pytest.mark.parametrize("mode", ["fp32", "bf16x3"])
def test_as_one_block_at_a_time(sv, n, batch, count, widths, low, rows, mode):
    rng = np.random.default_rng(7 * n + count)
    m = sv.FUSED_FP32_MFMA if mode == "fp32" else sv.FUSED_BF16X3
    if mode == "fp32":
        widths = tuple(w for w in widths if w < 6)
    blocks = _blocks(n, count, rng, widths, range(10) if low else None, batch if rows else 0)
    psi = np.stack([pins.random_state(n, rng) for _ in range(batch)]).astype(np.complex64)
    got = _run(sv, n, batch, psi, [blocks], m, rows)
    want = _run(sv, n, batch, psi, [[b] for b in blocks], m, rows)
    if mode == "bf16x3":
        assert np.array_equal(got, want)
    else:
        assert np.linalg.norm(got - want) <= 1e-7 * count * np.linalg.norm(want)
