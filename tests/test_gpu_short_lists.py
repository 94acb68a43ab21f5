"""Lists of a few gates, which go as sweeps of their own or share one: every kind
with up to three controls on low and high qubits, matrices of every row, explicit
matrices that are not unitary, against the oracle, on sizes around the rule's
lines; the adjoint of such lists; a captured list replayed.

Tolerance: 1e-5 absolute on amplitudes of a normalised state (as the other gate
tests); a matrix that is not unitary scales it by its norm."""

import numpy as np
import pytest

import oracle
from paper_2511_19291_amd import circuits as C
from tests import pins

pytestmark = pytest.mark.gpu

AMP_TOL = 1e-5


@pytest.mark.parametrize("n, batch, lists", [(4, 1, 60), (5, 3, 40), (9, 1, 40), (12, 2, 30), (15, 1, 30), (16, 1, 30),
                                             (16, 4, 12), (19, 1, 12), (20, 1, 8), (21, 1, 6), (22, 1, 4)])
def test_matches_oracle(sv, n, batch, lists):
    rng = np.random.default_rng(n + 100 * batch)
    psi = pins.random_state(n, rng).astype(np.complex64)
    st = sv.State(n, batch)
    for i in range(lists):
        circ = C.random_circuit(n, 2 + i % 4, 5000 + 100 * n + i, max_controls=3)
        rows = np.tile(circ.params, (batch, 1))
        if i % 2 and circ.n_params:
            rows = rng.uniform(0, 2 * np.pi, size=rows.shape)
        st.from_numpy(np.tile(psi, (batch, 1)))
        out = st.run(circ, params=rows if batch > 1 else rows[0]).to_numpy()
        for r in range(batch):
            ref = psi.astype(np.complex128)
            oracle.run(C.Circuit(n, circ.ops, rows[r]), psi=ref)
            assert np.max(np.abs(out[r] - ref)) <= AMP_TOL, (i, circ.ops)


@pytest.mark.parametrize("n", [4, 11, 13, 18])
def test_matrices_that_are_not_unitary(sv, n):
    rng = np.random.default_rng(n)
    psi = pins.random_state(n, rng).astype(np.complex64)
    st = sv.State(n)
    for count in (2, 3, 7):
        ops, mats = [], {}
        ref = psi.astype(np.complex128)
        for i in range(count):
            k = 1 + int(rng.integers(2))
            w = [int(q) for q in rng.permutation(n)]
            m = rng.normal(size=(1 << k, 1 << k)) + 1j * rng.normal(size=(1 << k, 1 << k))
            if i % 3 == 1:
                m = np.diag(np.diag(m))
            ops.append(C.Op("matrix", tuple(w[:k]), tuple(w[k:k + int(rng.integers(2))]), ()))
            mats[i] = m
            oracle.apply_matrix(ref, n, m, list(ops[-1].targets), list(ops[-1].controls))
        st.from_numpy(psi[None])
        st.run_ops(sv.OpTable(ops, mats), 0, count, np.zeros(0))
        assert np.max(np.abs(st.to_numpy()[0] - ref)) <= AMP_TOL * max(1.0, np.linalg.norm(ref))


@pytest.mark.parametrize("n, batch", [(4, 2), (13, 1), (16, 3), (18, 1)])
def test_adjoint_of_short_lists(sv, n, batch):
    rng = np.random.default_rng(7 * n)
    terms = C.z_sum_terms(n) + [C.pauli_term(0.5, "X0 Y1")]
    st = sv.State(n, batch)
    for i in range(6):
        b = C._Builder(n)
        for q in rng.permutation(n)[:3]:
            b.gate("ry", [int(q)], values=[rng.uniform(0.3, 2.8)])
        for j in range(2 + i % 3):
            w = [int(q) for q in rng.permutation(n)]
            if j % 2:
                b.gate("rx", [w[0]], w[1:1 + int(rng.integers(3))], [rng.uniform(0, 6)])
            else:
                b.gate(("x", "z", "h")[int(rng.integers(3))], w[:1], w[1:1 + int(rng.integers(4))])
        circ = b.build("short")
        rows = rng.uniform(0.3, 2.8, size=(batch, circ.n_params))
        params = rows if batch > 1 else rows[0]
        st.reset().run(circ, params=params)
        loss, grad, drift = st.adjoint_grad(circ, terms, params=params)
        assert np.max(drift) < 1e-4
        for r in range(batch):
            want, ref, _ = oracle.grad_adjoint(circ, terms, rows[r])
            assert abs(loss[r] - want) < 1e-4
            assert np.linalg.norm(grad[r] - ref) <= 1e-4 * max(np.linalg.norm(ref), 1.0)


def test_captured_short_list_replays(sv):
    import torch

    n = 18
    b = C._Builder(n)
    b.gate("h", [0])
    b.gate("x", [17], [0, 5, 9])
    circ = b.build("two")
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        st = sv.State(n)
        want = st.reset().run(circ).to_numpy()
        graph = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            st.reset().run(circ)
        for k in range(3):
            st.reset(k).run(circ)
            torch.cuda.synchronize()
            graph.replay()
            stream.synchronize()
            assert np.array_equal(st.to_numpy(), want)
