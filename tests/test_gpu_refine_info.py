"""What a refinement reports belongs to the solution that it returns: when the
last correction does not lower the backward error and is dropped, eta and
rel_residual are those of the iterate kept, bit for bit what a run that stops
there reports (the passes are deterministic)."""
import numpy as np
import pytest

import paper_2605_13736_amd as mds
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_d,n_s,m,sblk", [(40, 500, 80, 0), (100, 3000, 300, 0), (300, 0, 0, 0),
                                            (40, 500, 80, 4)])
def test_info_of_a_rejected_step(n_d, n_s, m, sblk):
    prob = synth.make_problem(n_d, n_s, m, 4 if n_s else 0, cfg=77, sblk=sblk)
    st = synth.kkt_state(prob, 1, (-3.0, 3.0))
    print(f"[gpu-case] refine info n_d={n_d} m={m} sblk={sblk}", flush=True)
    S = mds.solver_for(prob)
    S.condense(st["sigma_d"], st["dsbase"], 0.0, 0.0)
    S.factor_inertia()
    runs, rejected = [], 0
    for k in range(8):
        x, info = S.refine(st["r_d"], st["r_s"], st["r_y"], k, 0.0)
        runs.append((info, np.concatenate([t.cpu().numpy() for t in x])))
        if k and info["eta"] == runs[k - 1][0]["eta"] and np.array_equal(runs[k][1], runs[k - 1][1]):
            assert info["rel_residual"] == runs[k - 1][0]["rel_residual"]
            rejected += 1
    # at eta_tol = 0 the error cannot fall eight times
    assert rejected > 0
