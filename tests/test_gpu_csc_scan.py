"""Column-compressed copy of J_s at sizes around the scan's rounds of 8192
columns: the condensed matrix, which is summed through it, equals the oracle's bit
for bit (the same IEEE sequence), so every column pointer has to be right."""
import numpy as np
import pytest

import oracle
import paper_2605_13736_amd as mds
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns", [1, 7, 8, 63, 511, 8191, 8192, 8193, 16384, 40961])
def test_condense_through_the_copy(ns):
    print(f"[gpu-case] csc scan ns={ns}", flush=True)
    m = 48
    prob = synth.make_problem(5, ns, m, min(ns, 6), cfg=950, p=ns)
    st = synth.kkt_state(prob, 1, (-1.0, 1.0))
    S = mds.solver_for(prob)
    S.condense(st["sigma_d"], st["dsbase"], 0.0, 0.0)
    Mo, _ = oracle.condense(oracle.Problem(prob), st["sigma_d"], st["dsbase"], 0.0, 0.0)
    assert np.array_equal(S.get_matrix().view(np.int64), Mo.view(np.int64))
