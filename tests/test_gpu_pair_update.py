"""Two panels to one trailing update (large orders) against the look-ahead
factorization, whose trailing updates apply one panel each: the pivot
sequences agree and the solutions do within the rounding of the sums
(growth-bounded: 64 N eps relative to the larger solution entry times the
matrix's condition, which the diagonal keeps near one on the planted case).
The weak-diagonal matrix takes the second test on most steps, so the second
panel of a pair computes candidate columns outside its strip; the planted one
has failures at block, panel and pair edges only."""
import numpy as np
import pytest

import paper_2605_13736_amd as mds
from test_gpu_lookahead import _dense_problem, _weak_diag
from test_gpu_spec_panel import _planted

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,kind", [(6144, "weak"), (6273, "planted"), (6400, "planted")])
def test_pairs_match_single_updates(N, kind):
    print(f"[gpu-case] pair update N={N} {kind}", flush=True)
    if kind == "weak":
        A = _weak_diag(N, 5)
    else:
        A = _planted(N, [0, 15, 16, 62, 63, 64, 65, 126, 127, 128, 129, 191, 192, 300, 320, N - 17], 0, N)
    prob = _dense_problem(A)
    rhs = np.random.default_rng(N).standard_normal(N)
    out = []
    for la in ("off", "on"):
        S = mds.solver_for(prob, panel="coop", lookahead=la)
        assert (S.info()["lookahead_cus"] > 0) == (la == "on")
        S.condense(np.zeros(N), np.zeros(0), 0.0, 0.0)
        _, inn, _ = S.factor_inertia()
        piv = S.get_pivots().copy()
        (x, _, _), info = S.refine(rhs, np.zeros(0), np.zeros(0), 3, 1e-14)
        assert info["eta"] <= 64 * N * np.finfo(float).eps
        assert S.fallbacks()["coop_aborts"] == 0
        out.append((piv, (inn["npos"], inn["nzero"], inn["nneg"]), x.cpu().numpy()))
        del S
    assert np.array_equal(out[0][0], out[1][0])
    assert out[0][1] == out[1][1]
    if kind == "planted":
        d = np.abs(out[0][2] - out[1][2]).max()
        assert d <= 64 * N * np.finfo(float).eps * np.abs(out[0][2]).max()
