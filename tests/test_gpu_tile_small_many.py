"""States smaller than a tile in batches beyond two workgroups per compute unit
(513 rows and more), where a thread holds 16 amplitudes instead of 8: against the
oracle, with parameters shared and of every row.

Tolerance: 1e-5 absolute on amplitudes of a normalised state (as the other gate
tests)."""

import numpy as np
import pytest

import oracle
from paper_2511_19291_amd import circuits as C

pytestmark = pytest.mark.gpu

AMP_TOL = 1e-5


@pytest.mark.parametrize("n, batch", [(4, 513), (4, 4096), (5, 600), (7, 1025), (8, 700), (10, 520), (11, 514), (12, 513)])
def test_run_matches_oracle(sv, n, batch):
    circ = C.random_circuit(n, 120, 2000 + n)
    rng = np.random.default_rng(n)
    rows = np.tile(circ.params, (batch, 1))
    own = rng.random(circ.n_params) < 0.3
    rows[:, own] = rng.uniform(0, 2 * np.pi, size=(batch, int(own.sum())))
    picked = sorted({0, 1, 511, 512, batch // 2, batch - 1})
    st = sv.State(n, batch)
    out = st.reset().run(circ).to_numpy()
    ref = oracle.run(circ)
    for r in picked:
        assert np.max(np.abs(out[r] - ref)) <= AMP_TOL
    out = st.reset().run(circ, params=rows).to_numpy()
    for r in picked:
        assert np.max(np.abs(out[r] - oracle.run(C.Circuit(n, circ.ops, rows[r])))) <= AMP_TOL
    st.free()
