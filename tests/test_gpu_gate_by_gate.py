"""Gates handed over one at a time, each a sweep of its own (k_gate, k_diag): the
form behind sv_apply_gate, lone gates of a list and bench.py's timed step. Lists
share sweeps of tiles from four qubits on, so tests that hand over whole circuits
do not reach these kernels. The per-gate adjoint kernels (k_adj) run where a
two-target gate has a parameter.

Tolerances as in the tests of whole lists: 1e-5 absolute per amplitude
(complex64 against complex128, up to some hundred gates, each rounding once),
1e-4 relative for gradients; orders of the same sweep are equal to the bit."""

import json
import os

import numpy as np
import pytest
import torch

import oracle
from paper_2511_19291_amd import circuits as C
from tests import errmodel, pins

pytestmark = pytest.mark.gpu

AMP_TOL = 1e-5
GRAD_REL = 1e-4
KINDS_1Q = ["h", "x", "y", "z", "s", "sdg", "t", "tdg", "sx", "rx", "ry", "rz", "p", "u3"]
KINDS_2Q = ["swap", "rxx", "ryy", "rzz"]


def one_by_one(sv, st, circ):
    table = sv.OpTable(circ.ops)
    params = np.ascontiguousarray(circ.params)
    for i in range(len(circ.ops)):
        st.run_ops(table, i, 1, params)
    return st


def _uploaded(sv, n, seed, batch=1):
    psi = pins.random_state(n, np.random.default_rng(seed)).astype(np.complex64)
    return sv.State(n, batch).from_numpy(np.tile(psi, (batch, 1))), psi.astype(np.complex128)


@pytest.mark.parametrize("n", [4, 5, 6, 8, 9, 11, 13])
def test_every_kind_every_target(sv, n):
    """The float4, float2, pair-in-lane, shuffle and diagonal forms, qubit 0 and
    the top qubit among the targets, with no control and with one."""
    rng = np.random.default_rng(n)
    st, ref = _uploaded(sv, n, n)
    b = C._Builder(n)
    for kind in KINDS_1Q:
        for t in range(n):
            for ctrl in ([], [int(rng.integers(0, n))]):
                if ctrl and ctrl[0] == t:
                    continue
                b.gate(kind, [t], ctrl, rng.uniform(0, 2 * np.pi, C.N_PARAMS[kind]))
    for kind in KINDS_2Q:
        for t0 in range(n):
            for t1 in range(n):
                if t0 != t1:
                    b.gate(kind, [t0, t1], [], rng.uniform(0, 2 * np.pi, C.N_PARAMS[kind]))
    circ = b.build("all_kinds")
    out = one_by_one(sv, st, circ).to_numpy()[0]
    oracle.run(circ, psi=ref)
    assert np.max(np.abs(out - ref)) <= AMP_TOL


@pytest.mark.parametrize("n", [7, 12])
def test_low_qubit_access_forms(sv, n):
    """Controls and targets on the lowest qubits: the shuffle, odd-lane,
    pair-in-lane and masked-diagonal forms, and two-qubit gates at qubit 0."""
    rng = np.random.default_rng(40 + n)
    st, ref = _uploaded(sv, n, 40 + n)
    b = C._Builder(n)
    for t in range(1, n):
        b.gate("x", [t], [0])
        b.gate("z", [t], [0])
        b.gate("u3", [t], [0], rng.uniform(0, 2 * np.pi, 3))
        b.gate("p", [t], [0], [rng.uniform(0, 2 * np.pi)])
        b.gate("rz", [t], [0], [rng.uniform(0, 2 * np.pi)])
        b.gate("rxx", [0, t], [], [rng.uniform(0, 2 * np.pi)])
        b.gate("swap", [t, 0])
        b.gate("rzz", [t, 0], [], [rng.uniform(0, 2 * np.pi)])
    for t in range(1, min(7, n)):
        b.gate("u3", [t], [], rng.uniform(0, 2 * np.pi, 3))
        if t != n - 1:
            b.gate("ry", [t], [n - 1], [rng.uniform(0, 2 * np.pi)])
    b.gate("x", [0], [n - 1])
    b.gate("z", [0], [1, 2])
    circ = b.build("low_forms")
    out = one_by_one(sv, st, circ).to_numpy()[0]
    oracle.run(circ, psi=ref)
    assert np.max(np.abs(out - ref)) <= AMP_TOL


@pytest.mark.parametrize("n, seed", [(4, 1), (8, 2), (10, 3), (13, 4), (17, 5)])
def test_random_circuits(sv, n, seed):
    """Random kinds and targets with up to three controls."""
    circ = C.random_circuit(n, 200, seed, max_controls=3)
    out = one_by_one(sv, sv.State(n).reset(), circ).to_numpy()[0]
    assert np.max(np.abs(out - oracle.run(circ))) <= AMP_TOL


@pytest.mark.parametrize("n, batch", [(5, 3), (10, 4), (13, 2)])
def test_rows_with_their_own_parameters(sv, n, batch):
    circ = C.random_circuit(n, 60, 70 + n)
    rows = np.random.default_rng(n).uniform(0, 2 * np.pi, size=(batch, circ.n_params))
    st = sv.State(n, batch).reset()
    for op in circ.ops:
        st.run(C.Circuit(n, [op], circ.params), params=rows)
    out = st.to_numpy()
    for r in range(batch):
        assert np.max(np.abs(out[r] - oracle.run(C.Circuit(n, circ.ops, rows[r])))) <= AMP_TOL


def test_sweep_orders_equal_to_the_bit(sv):
    """The workgroup order of the one-target dense sweep changes which workgroup
    moves which pairs, never the arithmetic."""
    n = 14
    circ = C.brickwork_u3_cz(n, 4, 41)
    st = sv.State(n)
    saved = st.sweep_order()
    try:
        outs = []
        for mask in (0, (1 << n) - 1, 0b10101010101010):
            assert st.sweep_order(mask) == mask
            outs.append(one_by_one(sv, st.reset(), circ).to_numpy())
        for o in outs[1:]:
            assert np.array_equal(o.view(np.uint32), outs[0].view(np.uint32))
        assert np.max(np.abs(outs[1][0] - oracle.run(circ))) <= AMP_TOL
    finally:
        st.sweep_order(saved)
        st.free()


def test_gates_after_tuning_equal_the_hardware_order(sv):
    n, batch = 18, 2
    circ = C.brickwork_u3_cz(n, 3, 43)
    st = sv.State(n, batch)
    saved = st.sweep_order()
    try:
        st.reset().tune_sweep_order()
        a = one_by_one(sv, st.reset(), circ).to_numpy()
        st.sweep_order(0)
        b = one_by_one(sv, st.reset(), circ).to_numpy()
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))
        ref = oracle.run(circ)
        assert np.max(np.abs(a - ref)) <= AMP_TOL
    finally:
        st.sweep_order(saved)
        st.free()


def test_brickwork24_full_state(sv):
    circ = C.WORKLOADS["brickwork24"]()
    st = sv.State(24)
    out = one_by_one(sv, st.reset(), circ).to_numpy()[0].astype(np.complex128)
    st.free()
    ref = oracle.run(circ)
    d = out - ref
    assert np.max(np.abs(d)) <= AMP_TOL
    assert np.linalg.norm(d) <= errmodel.state_bound(errmodel.plain_circuit_eps(circ))


def test_brickwork30_as_bench_times_it(sv):
    """The step that bench.py times, a sweep per gate: <Z_i> and 1026 amplitudes
    against the oracle's stored values."""
    with open(os.path.join(os.path.dirname(__file__), "golden", "brickwork30.json")) as f:
        g = json.load(f)
    circ = C.WORKLOADS["brickwork30"]()
    st = one_by_one(sv, sv.State(30).reset(), circ)
    B = errmodel.state_bound(errmodel.plain_circuit_eps(circ))
    z = st.expval_z_all()[0]
    assert np.max(np.abs(z[:30] - np.array(g["expval_z"]))) <= errmodel.z_bound(B)
    idx = torch.as_tensor(np.asarray(g["amp_index"], dtype=np.int64), device=st.tensor.device)
    amps = st.tensor[0][idx].cpu().numpy().astype(np.complex128)
    ref = np.array(g["amp_re"]) + 1j * np.array(g["amp_im"])
    assert errmodel.sampled_norm_estimate(amps - ref, 30) <= B
    st.free()


@pytest.mark.parametrize("n", [4, 9, 13])
def test_adjoint_of_every_kind_and_target(sv, n):
    """One two-target gate with a parameter takes the whole backward gate by
    gate: every parameterised kind on every target, with and without a control."""
    rng = np.random.default_rng(300 + n)
    b = C._Builder(n)
    b.gate("rzz", [0, n - 1], [], [rng.uniform(0, 2 * np.pi)])
    for kind in ("rx", "ry", "rz", "p", "u3"):
        for t in range(n):
            c = int(rng.integers(0, n))
            b.gate(kind, [t], [] if c == t or c % 2 else [c], rng.uniform(0, 2 * np.pi, C.N_PARAMS[kind]))
            if t + 1 < n:
                b.gate("x", [t + 1], [t])
    for kind in ("rxx", "ryy", "rzz"):
        for t in range(n - 1):
            b.gate(kind, [t + 1, t] if t % 2 else [t, t + 1], [], [rng.uniform(0, 2 * np.pi)])
    circ = b.build("every_kind")
    terms = C.z_sum_terms(n) + [C.pauli_term(0.5, "X0 X1")]
    st = sv.State(n).reset().run(circ)
    loss, g, drift = st.adjoint_grad(circ, terms)
    want, ref, _ = oracle.grad_adjoint(circ, terms)
    assert np.linalg.norm(g[0] - ref) <= GRAD_REL * np.linalg.norm(ref)
    assert np.max(np.abs(g[0] - ref)) <= GRAD_REL * np.max(np.abs(ref))
    assert abs(loss[0] - want) < 1e-4 and drift[0] < 1e-4
