"""The Gaussian estimate and its weights from one set of sums, at the edges of
the sums' blocks of 2^12 amplitudes and rows of 256 workgroups x 4: one qubit,
one block, a block less and more, many blocks per workgroup; states at and near
the reflection's fixed basis vector (the last index), where its length is 0 or
small; weights written over the normals and to an array aligned to 8 bytes.

Tolerances: FP64 sums in another order than the oracle's, estimate 1e-10 and
weights 1e-9 of the largest. Near the last index the reflection divides by
R = 1e-4, which leaves FP64's 1e-16 three orders below both."""

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


def _check(sv, psi, n, shots, seed, out=None):
    rng = np.random.default_rng(seed)
    st = sv.State(n).from_numpy(psi.astype(np.complex64))
    ref = st.to_numpy()[0].astype(np.complex128)
    z = rng.normal(size=1 << n)
    g = rng.normal(size=n)
    zt = torch.tensor(z, device="cuda")
    np.testing.assert_allclose(st.gaussian_expval_z(zt, shots), oracle.gaussian_z(ref, n, z, shots), atol=1e-10)
    want = oracle.gaussian_z_weights(ref, n, z, shots, g)
    tol = {"rtol": 1e-9, "atol": 1e-9 * np.max(np.abs(want))}
    w = st.gaussian_expval_z_backward(zt, shots, g).cpu().numpy()
    np.testing.assert_allclose(w, want, **tol)
    room = torch.zeros((1 << n) + 1, dtype=torch.float64, device="cuda")[1:]
    st.gaussian_expval_z_backward(zt, shots, g, out=room)
    assert np.array_equal(room.cpu().numpy(), w)
    st.gaussian_expval_z_backward(zt, shots, g, out=zt)
    assert np.array_equal(zt.cpu().numpy(), w)


@pytest.mark.parametrize("n", [1, 2, 9, 11, 12, 13, 18, 23])
def test_random_states(sv, n):
    rng = np.random.default_rng(n)
    psi = rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)
    psi[rng.random(1 << n) < 0.01] = 0.0
    psi[0] += 1.0
    _check(sv, psi / np.linalg.norm(psi), n, 1e5, n)


@pytest.mark.parametrize("n, at, rest", [(3, 7, 0.0), (13, 8191, 0.0), (13, 0, 0.0), (6, 63, 1e-2), (14, 16383, 1e-2)])
def test_states_near_a_basis_vector(sv, n, at, rest):
    rng = np.random.default_rng(n)
    psi = rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)
    psi *= rest / np.linalg.norm(psi)
    psi[at] = 1.0
    _check(sv, psi, n, 1e5, n)
