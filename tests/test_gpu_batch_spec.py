"""FP64 scenario batch over speculative panels (4 nb columns, 8 nb from N = 1024 on): sizes at
the edges of a block, a 64-row group, a panel and a thread's row count, panel
widths that are no multiple of a block, and barrier states whose first test
fails often.  Bars: the oracle's inertia, trials and shift, and its solution
within 1e-8 (the tolerance of the linear solves)."""
import numpy as np
import pytest

import oracle
import paper_2605_13736_amd as mds
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb", [0, 3, 5, 16])
@pytest.mark.parametrize("spread", [1.0, 4.0])
def test_batch_edges_match_oracle(nb, spread):
    sizes = [4, 15, 16, 17, 63, 64, 65, 127, 129, 260, 511, 513, 600]
    if nb in (0, 5):
        sizes += [1025]
    print(f"[gpu-case] batch edges nb={nb} spread={spread}", flush=True)
    items, states = [], []
    for p, N in enumerate(sizes):
        nd = max(1, N // 4)
        prob = synth.make_problem(nd, 12 * N, N - nd, 3, cfg=840, p=p, s_scale=2.0)
        st = synth.kkt_state(prob, p, (-spread, spread))
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
