"""Exact draws with and without the sums of 16 amplitudes where the two can be
compared, and against the cumulative sum where they cannot. The sums are kept from
a draw per 880 amplitudes on, so up to 2^10 amplitudes by every call: those
states are checked against a search of the cumulative probabilities. On larger
ones every uniform, the ones on amplitudes' boundaries included, is drawn once
among all (with the sums) and once among a few (without)."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _state(sv, n):
    rng = np.random.default_rng(n)
    psi = rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)
    psi[rng.random(1 << n) < 0.2] = 0.0
    psi[1 << (n - 1):(1 << (n - 1)) + 40] = 0.0
    st = sv.State(n).from_numpy((psi / np.linalg.norm(psi)).astype(np.complex64))
    v = st.to_numpy()[0]
    return st, v.real.astype(np.float64) ** 2 + v.imag.astype(np.float64) ** 2, rng


@pytest.mark.parametrize("n", [7, 8, 9, 10])
def test_small_states_against_the_cumulative_sum(sv, n):
    """Uniforms at least 1e-9 of the norm away from every boundary: both sides'
    running sums are in 64 bits and off by some 1e-15."""
    st, p, rng = _state(sv, n)
    cum = np.cumsum(p) / p.sum()
    u = rng.random(3000)
    u = u[np.min(np.abs(u[:, None] - cum[None, :]), axis=1) > 1e-9]
    assert len(u) > 2900
    got = st.sample_exact(u).cpu().numpy()
    assert np.array_equal(got, np.searchsorted(cum, u, side="right"))
    assert np.array_equal(st.sample_exact(u[:1]).cpu().numpy(), got[:1])


@pytest.mark.parametrize("n, few", [(11, 1), (12, 3), (13, 8), (15, 36), (18, 296)])
def test_the_two_forms_agree_on_every_uniform(sv, n, few):
    assert few == (1 << n) // 880 - 1                 # the most draws without the sums
    st, p, rng = _state(sv, n)
    edges = np.cumsum(p)[rng.integers(0, 1 << n, 200)] / p.sum()
    u = np.clip(np.concatenate([rng.random(400), edges, np.nextafter(edges, 0.0), [0.0, 1.0 - 1e-16]]), 0.0, 1.0 - 1e-16)
    many = st.sample_exact(u).cpu().numpy()
    part = np.concatenate([st.sample_exact(u[i:i + few]).cpu().numpy() for i in range(0, len(u), few)])
    assert np.array_equal(many, part)
    assert np.all(p[many] > 0)
