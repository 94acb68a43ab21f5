"""Z estimates from given draw indices: draws without an index (-1), one draw,
counts around a wave, a workgroup and the draws a thread takes at once (15, with
two workgroups of 256 threads per CU), bits 0 and n - 1. Counts are integers, so
the estimates are equal to the host's."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, shots", [(1, 1), (3, 63), (5, 65), (12, 257), (20, 256 * 512 * 2 + 1),
                                      (9, 256 * 512 * 15 + 77), (27, 1 << 20)])
def test_counts_are_exact(sv, n, shots):
    rng = np.random.default_rng(shots)
    idx = rng.integers(0, 1 << n, shots)
    idx[rng.random(shots) < 0.1] = -1
    idx[0] = (1 << n) - 1
    got = sv.State(n).sample_z_estimate(idx).cpu().numpy()
    ok = idx[idx >= 0]
    want = [1.0 - 2.0 * (float(np.count_nonzero((ok >> q) & 1)) / float(ok.size)) for q in range(n)]
    assert np.array_equal(got, want)
