"""FP64 scenario batch from N = 1024 on, whose panels take 8 nb <= 128 columns:
orders at the rule's edge and at block, part and panel edges, with the failing
pivots (they gather where n_d ends) in either half of a panel, so that
interchanges reach back over more than 64 columns.  Bars: the oracle's inertia,
trials and shift, and its solution within 1e-8 (the tolerance of the linear
solves)."""
import numpy as np
import pytest

import oracle
import paper_2605_13736_amd as mds
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb", [16, 9])
def test_wide_panels_match_oracle(nb):
    print(f"[gpu-case] batch wide nb={nb}", flush=True)
    items, states = [], []
    for p, (N, nd) in enumerate([(1023, 240), (1024, 100), (1024, 230), (1089, 320), (1152, 500)]):
        prob = synth.make_problem(nd, 12 * N, N - nd, 3, cfg=870, p=p, s_scale=2.0)
        st = synth.kkt_state(prob, p, (-4.0, 4.0))
        items.append(dict(prob, **st))
        states.append((prob, st))
    B = mds.Batch(items, nb=nb)
    res = B.run(1e-2)
    for p, (prob, st) in enumerate(states):
        F = oracle.Factor(oracle.Problem(prob))
        F.correct(st["sigma_d"], st["dsbase"], 1e-2)
        assert res[p]["inertia"] == F.inertia == (prob["n_d"], 0, prob["m"])
        assert res[p]["trials"] == F.s.trials and res[p]["delta_w"] == F.s.dw
        ref = np.concatenate(F.solve(st["r_d"], st["r_s"], st["r_y"])[:3])
        got = np.concatenate(B.solution(p))
        assert np.abs(got - ref).max() <= 1e-8 * np.abs(ref).max()
