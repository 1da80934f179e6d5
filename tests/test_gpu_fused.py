"""Fused passes over the rows of the Newton system: sizes at the edges of the
row blocks (16 x_d rows, 64 y rows, 1024 x_s entries), empty parts and
inequality rows.  Bars against the oracle: a dot product of n terms differs by
at most n eps of its terms' magnitude, so every value is compared within
4 n eps of the sum of magnitudes that forms it, n = n_d + n_s + m + 8 (the
barrier terms and the scale factors)."""
import numpy as np
import pytest

import oracle
import paper_2605_13736_amd as mds
import synth
from helpers import full_kkt
from test_gpu_ineq import _interior

pytestmark = pytest.mark.gpu
EPS = np.finfo(float).eps

CASES = [(1, 0, 1, 0, 0), (15, 1, 0, 0, 0), (16, 63, 1, 1, 0), (17, 64, 63, 3, 0), (64, 1023, 64, 4, 7),
         (65, 1024, 65, 4, 65), (0, 1025, 40, 3, 0), (129, 5000, 130, 5, 1), (1030, 300, 257, 2, 100)]


def _np(t):
    return t.detach().cpu().numpy()


@pytest.mark.parametrize("nd,ns,m,r,mI", CASES)
def test_values_and_refinement(nd, ns, m, r, mI):
    print(f"[gpu-case] fused nd={nd} ns={ns} m={m} r={r} mI={mI}", flush=True)
    prob = synth.make_problem(nd, ns, m, r, cfg=900 + nd, m_I=mI) if mI else \
        synth.make_problem(nd, ns, m, r, cfg=900 + nd)
    if mI:
        x, y, zl, zu, mu = _interior(prob, 3)
    else:
        it = synth.interior_iterate(prob, 3)
        x, y, zl, zu, mu = it["x"], it["y"], it["zl"], it["zu"], it["mu"]
    P = oracle.Problem(prob)
    n = nd + ns
    tol = 4 * (n + m + 8) * EPS
    S = mds.solver_for(prob)
    K = full_kkt(prob, np.zeros(nd), prob["w"])   # [H, w, J] without shifts
    A = np.abs(K)
    ax = np.abs(np.concatenate([x[:n], np.zeros(m)]))
    ay = np.abs(np.concatenate([np.zeros(n), y]))
    hx, jy = (A @ ax)[:n], (A @ ay)[:n]
    cg = np.abs(np.concatenate([prob["c"], prob["g"]]))
    rows = (A @ ax)[n:] + np.abs(prob["b"])
    if mI:
        rows[m - mI:] += np.abs(x[n:])
    logs = 50.0 * len(x)   # |log| of a slack in [e-50, e50]
    f, phi, th = S.merit(x, mu)
    fs = float(ax[:n] @ (0.5 * hx + cg))
    assert abs(f - oracle.objective(P, x)) <= tol * fs
    assert abs(phi - oracle.barrier(P, x, mu)) <= tol * (fs + mu * logs)
    assert abs(th - oracle.theta(P, x)) <= tol * max(rows.sum(), 1e-300)
    E, _ = S.opt_error(x, y, zl, zu, mu)
    Eo, _ = oracle.opt_error(P, x, y, zl, zu, mu)
    scale = max(np.max(hx + jy + cg, initial=0.0) + np.abs(zl).max(initial=0) +
                np.abs(zu).max(initial=0), rows.max(initial=0.0), Eo)
    assert abs(E - Eo) <= tol * scale
    st = synth.kkt_state(prob, 3, (-1.0, 1.0))
    S.condense(st["sigma_d"], st["dsbase"], 0.0, 1e-6)
    S.factor_inertia()
    (dd, ds, dy), info = S.refine(st["r_d"], st["r_s"], st["r_y"], 3, 1e-14)
    F = full_kkt(prob, st["sigma_d"], st["dsbase"], 0.0, 1e-6)
    d = np.concatenate([_np(dd), _np(ds), _np(dy)])
    rhs = np.concatenate([st["r_d"], st["r_s"], st["r_y"]])
    res = np.abs(rhs - F @ d).max()
    eta = res / (np.abs(F).sum(1).max() * np.abs(d).max() + np.abs(rhs).max())
    assert abs(info["eta"] - eta) <= tol
    assert eta <= 1e-13
    assert abs(info["rel_residual"] * np.abs(rhs).max() - res) <= tol * (
        np.abs(F) @ np.abs(d) + np.abs(rhs)).max()
