"""The automatic choice moves between the cooperative panel, which is fast while
the pivots pass the first Bunch-Kaufman test, and the register panel, whose
pivots cost the same whatever the test says.  Matrices that fail it on most
steps, in their first or last part only, or in stripes (more changes than are
allowed): the oracle's pivots and inertia, a solve within the rounding of its
sums (64 N eps), and few steps of the cooperative panel on the failing ones."""
import numpy as np
import pytest

import oracle
import paper_2605_13736_amd as mds

pytestmark = pytest.mark.gpu


def _dense_problem(A):
    N = A.shape[0]
    return dict(n_d=N, n_s=0, m=0, r=0, H=np.asfortranarray(A), c=np.zeros(N), w=np.zeros(0),
                g=np.zeros(0), Jd=np.zeros((0, N)), rp=np.zeros(1, dtype=np.int32),
                ci=np.zeros(0, dtype=np.int32), v=np.zeros(0), b=np.zeros(0),
                xl=-np.ones(N), xu=np.ones(N))


def _matrix(N, kind):
    rng = np.random.default_rng(3 * N + len(kind))
    A = rng.standard_normal((N, N))
    A = 0.5 * (A + A.T)
    i = np.arange(N)
    A[i, i] *= 0.01
    strong = {"weak": i < 0, "head": i >= N // 2, "tail": i < N // 2, "stripes": i // 40 % 2 == 1,
              "zeros": i < 0}[kind]
    A[i[strong], i[strong]] = np.where(rng.random(strong.sum()) < 0.5, 1.0, -1.0) * 1e6
    if kind == "zeros":
        A[i % 23 == 5] = 0.0
        A[:, i % 23 == 5] = 0.0
    return A


CASES = [(N, kind, 0) for N in (40, 101, 257, 300, 513, 1025)
         for kind in ("weak", "head", "tail", "stripes", "zeros")]
CASES += [(300, "stripes", 2), (300, "head", 7), (513, "weak", 16), (2048, "stripes", 0),
          (2112, "weak", 0), (2112, "head", 33)]


@pytest.mark.parametrize("N,kind,nb", CASES)
def test_panel_switch_pivots(N, kind, nb):
    A = _matrix(N, kind)
    print(f"[gpu-case] panel switch N={N} {kind} nb={nb}", flush=True)
    S = mds.solver_for(_dense_problem(A), nb=nb)
    assert S.info()["panel"] == "coop"
    _, dd, ds, ipo, _, _ = oracle.bk(A)
    io = tuple(oracle.inertia(ipo, dd, ds)[:3])
    for timing in (False, True, False):  # captured and plain launches
        S.set_timing(timing)
        S.condense(np.zeros(N), np.zeros(0), 0.0, 0.0)
        _, inn, _ = S.factor_inertia()
        assert np.array_equal(S.get_pivots(), ipo)
        assert (inn["npos"], inn["nzero"], inn["nneg"]) == io
        if timing:
            tim = S.get_timings()
            assert tim["factor"]["launches"] == 1
            if N > 2000 and kind == "weak":  # changed by the host
                assert tim["panel_tail"]["launches"] > 0
    assert S.fallbacks()["coop_aborts"] == 0
    if N > 200 and nb == 0 and kind in ("weak", "zeros"):
        assert S.panel_stats()["coop_steps"] < max(N - 2048, 0) + 100
    if inn["nzero"] == 0:
        r = np.random.default_rng(N).standard_normal(N)
        x = S.solve(r, np.zeros(0), np.zeros(0))[0].cpu().numpy()
        eps = np.finfo(float).eps
        scale = np.abs(A).sum(1).max() * np.abs(x).max() + np.abs(r).max()
        assert np.abs(A @ x - r).max() <= 64 * N * eps * scale


@pytest.mark.parametrize("N,kind", [(257, "weak"), (600, "stripes"), (1200, "head")])
def test_panel_switch_mixed_precision(N, kind):
    A = _matrix(N, kind)
    print(f"[gpu-case] panel switch fp32 N={N} {kind}", flush=True)
    S = mds.solver_for(_dense_problem(A), precision="fp32")
    S.condense(np.zeros(N), np.zeros(0), 0.0, 0.0)
    S.factor_inertia()
    r = np.random.default_rng(N).standard_normal(N)
    (x, _, _), info = S.refine(r, np.zeros(0), np.zeros(0), 60, 1e-13)
    assert info["eta"] <= 1e-12
    x = x.cpu().numpy()
    res = np.abs(A @ x - r).max()
    assert res <= 2e-12 * (np.abs(A).sum(1).max() * np.abs(x).max() + np.abs(r).max())


def test_passing_pivots_stay_on_the_cooperative_panel():
    N = 700
    A = _matrix(N, "tail")
    A[np.arange(N), np.arange(N)] = 1e6
    S = mds.solver_for(_dense_problem(A))
    S.condense(np.zeros(N), np.zeros(0), 0.0, 0.0)
    S.factor_inertia()
    st = S.panel_stats()
    assert st["coop_steps"] == N and st["coop_second"] == 0


@pytest.mark.parametrize("N,precision", [(300, "fp64"), (771, "fp64"), (2048, "fp64"), (600, "fp32")])
def test_expired_wait_goes_to_the_register_panel(N, precision):
    # up to 2048 rows the one-workgroup panel, which waits for nobody, factors
    # what an expired exchange wait left; the next factorization does not try
    # the exchange at once
    A = _matrix(N, "head")
    print(f"[gpu-case] expired wait N={N} {precision}", flush=True)
    S = mds.solver_for(_dense_problem(A), precision=precision)
    _, dd, ds, ipo, _, _ = oracle.bk(A)
    io = tuple(oracle.inertia(ipo, dd, ds)[:3])
    S.set_timing(True)
    S.set_debug(mds.MDS_DEBUG_COOP_ABORT)
    aborts = []
    for _ in range(5):
        before = S.get_timings()["panel_tail"]["launches"]
        S.condense(np.zeros(N), np.zeros(0), 0.0, 0.0)
        _, inn, _ = S.factor_inertia()
        assert (inn["npos"], inn["nzero"], inn["nneg"]) == io
        if precision == "fp64":
            assert np.array_equal(S.get_pivots(), ipo)
        assert S.get_timings()["panel_tail"]["launches"] - before >= N // 32
        aborts.append(S.fallbacks()["coop_aborts"])
    assert aborts == [1, 1, 2, 2, 2]
    r = np.random.default_rng(N).standard_normal(N)
    (x, _, _), info = S.refine(r, np.zeros(0), np.zeros(0), 60, 1e-13)
    assert info["eta"] <= 1e-12
    S.set_debug(0)
    for _ in range(3):
        S.condense(np.zeros(N), np.zeros(0), 0.0, 0.0)
        S.factor_inertia()
    assert S.fallbacks()["coop_aborts"] == 2 and S.panel_stats()["coop_steps"] > 0
