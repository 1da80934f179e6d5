"""Condensation with rows of J_s of 0 to 9 entries (the Schur kernel reads four
entries together) that share most of their columns: M and D_s^{-1} bit for bit
the oracle's."""
import numpy as np
import pytest

import oracle
import paper_2605_13736_amd as mds
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_d,n_s,m", [(3, 9, 1), (5, 12, 40), (0, 30, 129), (64, 2000, 128)])
@pytest.mark.parametrize("first", [0, 3, 4, 7])
def test_ragged_rows(n_d, n_s, m, first):
    prob = synth.make_problem(n_d, n_s, m, 2, cfg=402)
    rng = np.random.default_rng(n_s + first)
    ln = (first + np.arange(m)) % 10
    prob["rp"] = np.concatenate([[0], np.cumsum(ln)]).astype(np.int32)
    prob["ci"] = np.concatenate([np.sort(rng.choice(n_s, k, replace=False)) for k in ln]).astype(np.int32)
    prob["v"] = rng.standard_normal(int(ln.sum()))
    sd, db = rng.uniform(0.5, 2.0, n_d), rng.uniform(0.1, 10.0, n_s)
    print(f"[gpu-case] ragged condense n_d={n_d} n_s={n_s} m={m} first={first}", flush=True)
    S = mds.solver_for(prob)
    S.condense(sd, db, 1e-6, 1e-9)
    Mo, invo = oracle.condense(oracle.Problem(prob), sd, db, 1e-6, 1e-9)
    assert np.array_equal(np.asarray(S.get_matrix()).view(np.int64), Mo.view(np.int64))
    assert np.array_equal(S.get_inv_ds().view(np.int64), invo.view(np.int64))
