"""Problems without rows: y is empty (a null pointer) and J'y is zero, in the
fused passes and in the separate ones of coupling blocks.  A whole IPM matches
the oracle's, whatever the workspace held before."""
import numpy as np
import pytest

import oracle
import paper_2605_13736_amd as mds
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_d,n_s,sblk", [(20, 40, 0), (64, 0, 0), (0, 50, 0), (20, 40, 4), (0, 60, 5),
                                          (40, 7, 3)])
def test_ipm_without_rows(n_d, n_s, sblk):
    import torch
    prob = synth.make_problem(n_d, n_s, 0, 0, cfg=77, sblk=sblk)
    o = oracle.ipm(oracle.Problem(prob))
    assert o["status"] == "converged"
    for k in range(3):
        print(f"[gpu-case] no rows n_d={n_d} n_s={n_s} sblk={sblk} {k}", flush=True)
        # the next workspace takes the memory of one filled with 32.5
        S = mds.solver_for(prob)
        S.ws.fill_(0x40)
        torch.cuda.synchronize()
        del S
        S = mds.solver_for(prob)
        r = S.ipm_solve()
        assert r["status"] == o["status"] and r["iters"] == o["iters"]
        x = r["x"].cpu().numpy()
        assert np.abs(x - o["x"]).max() <= 1e-8 * max(1.0, np.abs(o["x"]).max())
