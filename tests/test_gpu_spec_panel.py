"""Speculative blocks of the cooperative panel: matrices whose pivots pass the
first Bunch-Kaufman test except at planted positions (block, four-column and
panel edges, the matrix's ends), where each way out of a failure is taken
(second test, interchange, 2x2, zero pivot).  Bars: the oracle's pivot
sequence, inertia and info, and a solve whose backward error is within the
sum's rounding, 64 N eps (the planted rows bound the growth)."""
import numpy as np
import pytest

import oracle
import paper_2605_13736_amd as mds

pytestmark = pytest.mark.gpu


def _planted(N, where, kind, seed):
    rng = np.random.default_rng(seed)
    A = 0.02 * rng.standard_normal((N, N)) / max(1.0, np.sqrt(N) / 8)
    A = A + A.T
    A[np.arange(N), np.arange(N)] = np.where(rng.random(N) < 0.5, 1.0, -1.0) * rng.uniform(1, 2, N)
    for n, p in enumerate(x for x in where if x < N - 1):
        q = int(rng.integers(p + 1, N))
        how = (kind + n) % 3 if kind < 3 else n % 4
        if how == 0:      # 2x2 (or the second test): both diagonals small
            A[p, p], A[q, q] = 0.01, 0.02
            A[p, q] = A[q, p] = 3.0
        elif how == 1:    # interchange: the candidate's diagonal is large
            A[p, p], A[q, q] = 0.05, 9.0
            A[p, q] = A[q, p] = 2.0
        elif how == 2:    # second test: the candidate's own row is larger
            z = (q + 1) % N if (q + 1) % N > p else p + 1
            A[p, p], A[q, q] = 1.0, 0.1
            A[p, q] = A[q, p] = 2.0
            if z != q:
                A[z, q] = A[q, z] = 9.0
        else:             # a zero row and column
            A[p, :] = 0.0
            A[:, p] = 0.0
    return A


CASES = [(1, 0), (2, 0), (15, 0), (16, 0), (17, 0), (33, 7), (64, 0), (65, 16), (255, 0), (256, 0),
         (257, 0), (300, 17), (513, 0), (700, 0), (2049, 0), (2112, 0), (2300, 33)]


@pytest.mark.parametrize("kind", [0, 1, 2, 3])
@pytest.mark.parametrize("N,nb", CASES)
def test_planted_failures(N, nb, kind):
    print(f"[gpu-case] planted N={N} nb={nb} kind={kind}", flush=True)
    where = [0, 3, 4, 14, 15, 16, 31, 47, 62, 63, 64, 130, 255, 256, 300, N - 17, N - 2]
    A = _planted(N, sorted({p for p in where if 0 <= p}), kind, 7 * N + kind)
    prob = dict(n_d=N, n_s=0, m=0, r=0, H=np.asfortranarray(A), c=np.zeros(N), w=np.zeros(0),
                g=np.zeros(0), Jd=np.zeros((0, N)), rp=np.zeros(1, dtype=np.int32),
                ci=np.zeros(0, dtype=np.int32), v=np.zeros(0), b=np.zeros(0), xl=-np.ones(N),
                xu=np.ones(N))
    S = mds.solver_for(prob, nb=nb, panel="coop")
    S.condense(np.zeros(N), np.zeros(0), 0.0, 0.0)
    _, inn, _ = S.factor_inertia()
    _, dd, ds, ipo, info, _ = oracle.bk(A)
    assert np.array_equal(S.get_pivots(), ipo)
    io = oracle.inertia(ipo, dd, ds)
    assert (inn["npos"], inn["nzero"], inn["nneg"]) == tuple(io[:3])
    assert S.fallbacks()["coop_aborts"] == 0
    if inn["nzero"] == 0:
        r = np.random.default_rng(N).standard_normal(N)
        x = S.solve(r, np.zeros(0), np.zeros(0))[0].cpu().numpy()
        eps = np.finfo(float).eps
        scale = np.abs(A).sum(1).max() * np.abs(x).max() + np.abs(r).max()
        assert np.abs(A @ x - r).max() <= 64 * N * eps * scale
