"""Look-ahead on request past N = 16384, where the panel takes more than 64
compute units, and off by itself at every size."""
import numpy as np
import pytest

import paper_2605_13736_amd as mds
import synth

pytestmark = pytest.mark.gpu


def test_lookahead_past_16384_equals_sequential():
    prob = synth.make_problem(128, 60000, 16512, 4, cfg=360)  # N = 16640: 65 workgroups
    st = synth.kkt_state(prob, 1, (-2.0, 2.0))
    res = {}
    for la in ("auto", "on"):
        print(f"[gpu-case] N=16640 lookahead={la}", flush=True)
        S = mds.solver_for(prob, lookahead=la)
        assert (S.info()["lookahead_cus"] >= 65) == (la == "on")
        S.condense(st["sigma_d"], st["dsbase"], 0.0, 0.0)
        _, inn, _ = S.factor_inertia()
        x = np.concatenate([t.cpu().numpy() for t in S.solve(st["r_d"], st["r_s"], st["r_y"])])
        res[la] = (S.get_pivots(), inn, x)
        assert S.fallbacks()["coop_aborts"] == 0
        del S
    (p0, i0, x0), (p1, i1, x1) = res["auto"], res["on"]
    assert np.array_equal(p0, p1) and i0 == i1
    assert np.abs(x1 - x0).max() <= 1e-12 * np.abs(x0).max()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("N", [8192, 9000, 16640])
def test_lookahead_is_off_by_itself(N, precision):
    S = mds.Solver(128, 1000, N - 128, 4 * (N - 128), precision=precision)
    assert S.info()["lookahead_cus"] == 0
