"""Condensation with many sparse variables beside few dense rows, or none:
D_s^{-1} bit for bit and M's blocks against their definition."""
import numpy as np
import pytest

import paper_2605_13736_amd as mds
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_d,n_s,m", [(0, 1, 0), (0, 17_000_000, 0), (10, 200_000, 20), (1, 70_000, 0),
                                       (0, 300_001, 65), (64, 257, 0)])
def test_inverse_of_ds(n_d, n_s, m):
    prob = synth.make_problem(n_d, n_s, m, 3 if m else 0, cfg=401)
    rng = np.random.default_rng(n_s)
    sd, db = rng.uniform(0.5, 2.0, n_d), rng.uniform(0.1, 10.0, n_s)
    print(f"[gpu-case] condense n_d={n_d} n_s={n_s} m={m}", flush=True)
    S = mds.solver_for(prob)
    for dw in (0.0, 1e-3):
        S.condense(sd, db, dw, 0.0)
        inv = S.get_inv_ds()
        assert np.array_equal(inv, 1.0 / (db + dw))
        if n_d + m:
            M = np.asarray(S.get_matrix())
            A = prob["H"].copy()
            i = np.arange(n_d)
            A[i, i] = (A[i, i] + sd) + dw
            assert np.array_equal(M[:n_d, :n_d], A)
            assert np.array_equal(M[n_d:, :n_d], prob["Jd"])
