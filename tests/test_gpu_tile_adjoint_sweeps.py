"""The per-gate adjoint of states above 12 qubits in sweeps of a tile (one-target
parameters) against the oracle's adjoint: every one-target kind with up to
two controls inside and outside the tile, index maps whose controls lie outside,
parameters of every row, lists longer than one sweep or one launch's values,
observables with X and Y parts and given diagonals, run-to-run equality, the
recomputed start state.

Tolerance: relative error 1e-4 in norm and per component of the largest (the
stated gradient tolerance)."""

import numpy as np
import pytest
import torch

import oracle
from paper_2511_19291_amd import circuits as C
from tests.test_gpu_tile_adjoint import _circuit, _close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, gates, batch", [(13, 60, 1), (13, 500, 1), (14, 80, 3), (15, 120, 2), (16, 40, 20), (18, 90, 1)])
def test_matches_oracle(sv, n, gates, batch):
    circ = _circuit(n, gates, 10 * n + batch)
    rng = np.random.default_rng(n)
    rows = np.tile(circ.params, (batch, 1))
    own = rng.random(circ.n_params) < 0.4
    if batch > 1:
        rows[:, own] = rng.uniform(0, 2 * np.pi, size=(batch, int(own.sum())))
    terms = C.z_sum_terms(n)
    coeff = rng.normal(size=(batch, n))
    params = rows if batch > 1 else rows[0]
    st = sv.State(n, batch)
    got = []
    for _ in range(2):
        st.reset().run(circ, params=params)
        got.append(st.adjoint_grad(circ, terms, params=params, coeff_rows=coeff))
    for a, b in zip(*got):
        assert np.array_equal(a, b)
    loss, grad, drift = got[0]
    assert np.max(drift) < 1e-4
    for r in sorted({0, batch - 1}):
        mine = [(float(coeff[r, q]), x, z) for q, (_, x, z) in enumerate(terms)]
        want, ref, _ = oracle.grad_adjoint(circ, mine, rows[r])
        _close(grad[r], ref)
        assert abs(loss[r] - want) < 1e-4
    st.reset().run(circ, params=params)
    st.adjoint_grad(circ, terms, params=params, coeff_rows=coeff)
    assert np.max(np.abs(st.to_numpy() - np.eye(1, 1 << n))) < 1e-4       # the recomputed |0..0>


@pytest.mark.parametrize("name", ["rxry_ring", "ladder", "brickwork"])
def test_library_circuits(sv, name):
    n = 14
    circ = {"rxry_ring": lambda: C.rxry_ring(n, 3, 5), "brickwork": lambda: C.brickwork_u3_cz(n, 4, 5),
            "ladder": lambda: C.profiling_ladder(n, 2, 1, seed=5)[0]}[name]()
    terms = [C.pauli_term(0.6, "X0 Y13"), C.pauli_term(-1.0, "Z2 Z5"), C.pauli_term(0.4, "Z12")]
    st = sv.State(n).reset().run(circ)
    loss, grad, _ = st.adjoint_grad(circ, terms)
    want, ref, _ = oracle.grad_adjoint(circ, terms, circ.params)
    _close(grad[0], ref)
    assert abs(loss[0] - want) < 1e-4
    # a given diagonal: sum_i Z_i
    z = C.z_sum_terms(n)
    b = np.arange(1 << n)
    w = torch.tensor(sum(1.0 - 2.0 * ((b >> i) & 1) for i in range(n)), device="cuda").reshape(1, -1).contiguous()
    st.reset().run(circ)
    _, gd, _ = st.adjoint_grad_diag(circ, w)
    _, ref, _ = oracle.grad_adjoint(circ, z, circ.params)
    _close(gd[0], ref)
