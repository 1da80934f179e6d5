"""The panels against each other on dense random matrices, whose first test
fails on most steps: the automatic choice (which changes to the register panel
over the last 2048 rows), the cooperative panel to the end and the memory panel,
which share no panel code, give the same pivots and inertia and, up to rounding,
the same factor."""
import numpy as np
import pytest

import paper_2605_13736_amd as mds

pytestmark = pytest.mark.gpu


def _dense_problem(A):
    N = A.shape[0]
    return dict(n_d=N, n_s=0, m=0, r=0, H=np.asfortranarray(A), c=np.zeros(N), w=np.zeros(0),
                g=np.zeros(0), Jd=np.zeros((0, N)), rp=np.zeros(1, dtype=np.int32),
                ci=np.zeros(0, dtype=np.int32), v=np.zeros(0), b=np.zeros(0),
                xl=-np.ones(N), xu=np.ones(N))


@pytest.mark.parametrize("N", [257, 1024, 2049, 3000, 5000])
def test_panels_agree(N):
    rng = np.random.default_rng(N + 7)
    A = rng.standard_normal((N, N))
    A = A + A.T
    out = {}
    for panel in ("auto", "coop", "mem"):
        print(f"[gpu-case] dense N={N} panel={panel}", flush=True)
        S = mds.solver_for(_dense_problem(A), panel=panel)
        S.condense(np.zeros(N), np.zeros(0), 0.0, 0.0)
        _, inn, _ = S.factor_inertia()
        L, _, _, piv = S.get_factor()
        out[panel] = (L, piv, inn)
        assert S.fallbacks()["coop_aborts"] == 0
        if panel == "auto":
            assert 0 < S.panel_stats()["coop_steps"] < N // 2 or N > 4096
        del S
    L, piv, inn = out["mem"]
    for panel in ("auto", "coop"):
        assert np.array_equal(out[panel][1], piv), panel
        assert out[panel][2] == inn, panel
        # the same bar as the tests of the single panels
        assert np.abs(out[panel][0] - L).max() <= 1e-10 * max(1.0, np.abs(L).max()), panel
