"""Fused blocks of fewer than five qubits in a sweep with others: they are padded
with low qubits, which the sweep's tile may not hold (qubit 4, beside a block
within qubits 0..3). Against the blocks one call at a time, and in FP64.

Tolerance: BF16x3 equal to the bit to the single blocks; FP32 against FP64 in norm:
64 products of 2^-24 a block, 4e-6, at worst, six blocks; BF16x3 3 2^-16 more."""

import numpy as np
import pytest

from tests import pins

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("first", [[(0, 1, 2, 3)], [(3, 1, 0, 2)], [(2,)], [(1, 3), (0, 2)], [(3, 0, 1)]])
@pytest.mark.parametrize("mode", ["fp32", "bf16x3"])
def test_tile_without_qubit_four(sv, first, mode):
    n = 15
    rng = np.random.default_rng(sum(len(t) for t in first))
    m = sv.FUSED_FP32_MFMA if mode == "fp32" else sv.FUSED_BF16X3
    # nine qubits above the fourth fill the tile
    targets = list(first) + [(6, 7, 8, 9, 10), (11, 12, 13, 14)] + list(first) + [(14, 6)]
    blocks = [(t, pins.haar_unitary(1 << len(t), rng)) for t in targets]
    psi = pins.random_state(n, rng).astype(np.complex64)
    st = sv.State(n)
    got = st.from_numpy(psi[None]).apply_fused(blocks, m).to_numpy()[0]
    st.from_numpy(psi[None])
    for b in blocks:
        st.apply_fused([b], m)
    want = st.to_numpy()[0]
    ref = psi.astype(np.complex128)
    for t, u in blocks:
        # a block's unitary, whose first target is the most significant bit
        axes = [n - 1 - q for q in t]
        v = np.moveaxis(ref.reshape((2,) * n), axes, range(len(t)))
        w = (u @ v.reshape(1 << len(t), -1)).reshape(v.shape)
        ref = np.moveaxis(w, range(len(t)), axes).reshape(-1).copy()
    eps = 64 * 2.0 ** -24 + (3 * 2.0 ** -16 if mode == "bf16x3" else 0.0)
    assert np.linalg.norm(got - ref) <= eps * len(blocks) * np.linalg.norm(ref)
    if mode == "bf16x3":
        assert np.array_equal(got, want)
    else:
        assert np.linalg.norm(got - want) <= 1e-7 * len(blocks) * np.linalg.norm(want)
