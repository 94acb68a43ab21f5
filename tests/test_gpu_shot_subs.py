"""Exact draws with and without the sums of 16 amplitudes (many draws keep them,
few do not): the same uniforms give the same indices, drawn all at once and a
few at a time, on states of one small block, one chunk and several blocks, with
zero runs, and at uniforms on the boundaries of amplitudes."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, few", [(7, 1), (9, 1), (12, 3), (13, 8), (18, 290), (21, 2300)])
def test_same_indices(sv, n, few):
    rng = np.random.default_rng(n)
    psi = rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)
    psi[rng.random(1 << n) < 0.2] = 0.0
    psi[1 << (n - 1):(1 << (n - 1)) + 40] = 0.0
    st = sv.State(n).from_numpy((psi / np.linalg.norm(psi)).astype(np.complex64))
    p = np.abs(st.to_numpy()[0].astype(np.complex128)) ** 2
    edges = np.cumsum(p)[rng.integers(0, 1 << n, 50)] / p.sum()
    u = np.clip(np.concatenate([rng.random((1 << n) // 100 + 200), edges, [0.0, 1.0 - 1e-16]]), 0.0, 1.0 - 1e-16)
    many = st.sample_exact(u).cpu().numpy()
    # below a draw per 880 amplitudes: the chunks themselves are read
    part = np.concatenate([st.sample_exact(u[i:i + few]).cpu().numpy() for i in range(0, min(len(u), 60 * few), few)])
    assert np.array_equal(many[:len(part)], part)
    assert np.all(p[many] > 0)
    tail = st.sample_exact(u[-52:]).cpu().numpy() if n > 16 else many[-52:]
    assert np.array_equal(many[-52:], tail)
