"""Performance cases: what a program that uses this library has it do.

A case is one pass through the public entry points (``Solver``, ``Batch``,
``BatchIPM``, ``MLP``) on seeded synthetic problems of the repository's own
structure (mixed dense-sparse, H = Q Q'/n_d + S with S indefinite, r nonzeros
per row of J_s, bounds [-1, 1]).  Kinds:

* ``newton``: one Newton system of an interior-point step, condense + factor
  with the inertia-correction loop + refined solve.  ``decades`` is the spread
  of the barrier diagonals around 1 (Sigma = z / slack runs from mu to 1 / mu).
* ``ipm``: a whole interior-point solve from the cold start to E_0 <= 1e-8.
* ``batch``: many independent Newton systems in one persistent launch.
* ``batch_ipm``: many whole interior-point solves in one persistent launch.
* ``mlp_train`` / ``mlp_infer``: the warm-start perceptron (an epoch of
  training read back at its end; one inference call).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2605_13736_amd as mds

DEV = "cuda:0"
TINY = dict(kind="newton", n_d=37, n_s=900, m=64, r=4, decades=2, precision="fp64")


def listed():
    return [
        # a small controller-sized system: launch and latency bound
        dict(TINY, name="newton_n101"),
        # an odd mid-size system, one workgroup's panel
        dict(name="newton_n771", kind="newton", n_d=193, n_s=38000, m=578, r=4, decades=4,
             precision="fp64"),
        # an odd size just past the one-workgroup panel
        dict(name="newton_n2051", kind="newton", n_d=513, n_s=100003, m=1538, r=6, decades=2,
             precision="fp64"),
        # the OPF-scale Newton system (n_d = 1024, n_s = 200000, m = 3072)
        dict(name="newton_n4096", kind="newton", n_d=1024, n_s=200000, m=3072, r=6, decades=2,
             precision="fp64"),
        # the same system through the mixed-precision option (FP32 trailing
        # matrix, FP64 refinement)
        dict(name="newton_n4096_fp32", kind="newton", n_d=1024, n_s=200000, m=3072, r=6,
             decades=2, precision="fp32"),
        # a large odd system
        dict(name="newton_n9001", kind="newton", n_d=2257, n_s=500009, m=6744, r=8, decades=4,
             precision="fp64"),
        # the large condensed system (n_d = 4096, n_s = 10^6, m = 12288)
        dict(name="newton_n16384", kind="newton", n_d=4096, n_s=1000000, m=12288, r=8, decades=2,
             precision="fp64"),
        # a whole solve of the N = 192 problem (n_d = 64, n_s = 2000, m = 128)
        dict(name="ipm_n192", kind="ipm", n_d=64, n_s=2000, m=128, r=4, m_I=0),
        # a whole solve with inequality rows, odd size
        dict(name="ipm_n515_ineq", kind="ipm", n_d=129, n_s=5003, m=386, r=4, m_I=97),
        # the scenario batch (N = 256..2048 spread evenly over its range)
        dict(name="batch_512", kind="batch", count=512, n_lo=256, n_hi=2048, precision="fp64"),
        # whole solves of a batch of small scenarios
        dict(name="batch_ipm_256", kind="batch_ipm", count=256, n_lo=64, n_hi=320),
        # warm-start perceptron of the N = 192 family, an epoch of training
        dict(name="mlp_train_h256", kind="mlp_train", n_in=128, hidden=256, n_out=193, batch=64,
             steps=16),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["newton"] * 6 + ["ipm"] * 2 + ["batch", "batch_ipm", "mlp_train"])
    if kind == "newton":
        N = _log_int(rng, 90, 12000)
        n_d = max(2, int(N * rng.uniform(0.2, 0.4)))
        m = N - n_d
        mixed = rng.random() < 0.2
        return dict(kind=kind, n_d=n_d, n_s=int(m * rng.uniform(8.0, 60.0)), m=m,
                    r=rng.randint(4, 8), decades=2 if mixed else rng.randint(1, 4),
                    precision="fp32" if mixed else "fp64")
    if kind == "ipm":
        N = _log_int(rng, 64, 700)
        n_d = max(8, N // 4 + rng.randint(-3, 3))
        m = N - n_d
        return dict(kind=kind, n_d=n_d, n_s=m * rng.randint(10, 20), m=m, r=4,
                    m_I=rng.choice([0, m // 4]))
    if kind == "batch":
        lo = _log_int(rng, 64, 512)
        return dict(kind=kind, count=_log_int(rng, 16, 400), n_lo=lo, n_hi=lo * rng.randint(1, 4) + 3,
                    precision="fp64")
    if kind == "batch_ipm":
        return dict(kind=kind, count=_log_int(rng, 16, 256), n_lo=rng.randint(40, 80),
                    n_hi=rng.randint(100, 320))
    return dict(kind=kind, n_in=rng.randint(64, 700), hidden=32 * rng.randint(4, 12),
                n_out=rng.randint(64, 700), batch=rng.randint(16, 128), steps=16)


# ---- inputs ---------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(1 + int(seed))
    return g


def _problem(g, n_d, n_s, m, r, m_I=0):
    """One problem dict; dense blocks column-major, as the library takes them."""
    f = dict(device=DEV, dtype=torch.float64, generator=g)
    Q = torch.randn(n_d, n_d, **f)
    G = torch.randn(n_d, n_d, **f)
    # G + G' over sqrt(8 n): eigenvalues in [-1, 1] (semicircle)
    H = Q @ Q.T / n_d + (G + G.T) / math.sqrt(8.0 * n_d)
    H = 0.5 * (H + H.T)
    JdT = torch.randn(n_d, m, **f) / math.sqrt(n_d)
    # one column from each of r equal ranges of the sparse variables
    w = n_s // r
    cols = torch.randint(0, w, (m, r), device=DEV, generator=g) + w * torch.arange(r, device=DEV)
    vals = torch.randn(m, r, **f)
    x0 = torch.rand(n_d + n_s, **f) - 0.5
    b = JdT.T @ x0[:n_d] + (vals * x0[n_d:][cols]).sum(1)
    n = n_d + n_s
    hl = (b[m - m_I:] - 0.05 - 0.45 * torch.rand(m_I, **f)).cpu().numpy()
    hu = (b[m - m_I:] + 0.05 + 0.45 * torch.rand(m_I, **f)).cpu().numpy()
    return dict(n_d=n_d, n_s=n_s, m=m, m_I=m_I, H=H.cpu().numpy().T, Jd=JdT.cpu().numpy().T,
                c=torch.randn(n_d, **f).cpu().numpy(),
                w=(0.1 + 9.9 * torch.rand(n_s, **f)).cpu().numpy(),
                g=torch.randn(n_s, **f).cpu().numpy(),
                rp=np.arange(m + 1, dtype=np.int32) * r,
                ci=cols.reshape(-1).to(torch.int32).cpu().numpy(),
                v=vals.reshape(-1).cpu().numpy(), b=b.cpu().numpy(),
                xl=-np.ones(n), xu=np.ones(n), hl=hl, hu=hu)


def _barrier(g, prob, decades):
    """Barrier diagonals (Sigma_d, w + Sigma_s) and a right-hand side."""
    f = dict(device=DEV, dtype=torch.float64, generator=g)
    nd, ns, m = prob["n_d"], prob["n_s"], prob["m"]
    sd = 10.0 ** (decades * (2.0 * torch.rand(nd, **f) - 1.0))
    ss = 10.0 ** (decades * (2.0 * torch.rand(ns, **f) - 1.0))
    db = ss + torch.as_tensor(prob["w"], device=DEV)
    return dict(sigma_d=sd, dsbase=db, r_d=torch.randn(nd, **f), r_s=torch.randn(ns, **f),
                r_y=torch.randn(m, **f))


def _batch_problem(g, case, p):
    """Scenario p of a batch: N spread evenly over [n_lo, n_hi], n_d = N/4."""
    c = case["count"]
    N = case["n_lo"] + (case["n_hi"] - case["n_lo"]) * p // max(c - 1, 1)
    n_d = N // 4
    return _problem(g, n_d, 50 * N, N - n_d, 4)


def _mlp_data(case, seed):
    rng = np.random.default_rng(seed)
    n_in, h, n_out = case["n_in"], case["hidden"], case["n_out"]
    f32 = np.float32
    par = np.concatenate([
        rng.standard_normal(n_in * h).astype(f32) / f32(math.sqrt(n_in)), np.zeros(h, f32),
        rng.standard_normal(h * h).astype(f32) / f32(math.sqrt(h)), np.zeros(h, f32),
        rng.standard_normal(h * n_out).astype(f32) / f32(math.sqrt(h)), np.zeros(n_out, f32),
        rng.standard_normal(n_in * n_out).astype(f32) / f32(math.sqrt(n_in))])
    X = rng.standard_normal((case["steps"], case["batch"], n_in)).astype(f32)
    A = rng.standard_normal((n_in, n_out)).astype(f32) / f32(math.sqrt(n_in))
    return par, X, np.tanh(X @ A)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "mlp_train":
        net = mds.MLP((case["n_in"], case["hidden"], case["hidden"], case["n_out"]),
                      case["batch"])
        par, X, T = _mlp_data(case, seed)
        return dict(kind=kind, net=net, par=par, X=torch.as_tensor(X, device=DEV),
                    T=torch.as_tensor(T, device=DEV), steps=case["steps"])
    g = _gen(seed)
    if kind in ("newton", "ipm"):
        prob = _problem(g, case["n_d"], case["n_s"], case["m"], case["r"], case.get("m_I", 0))
        S = mds.solver_for(prob, precision=case.get("precision", "fp64"))
        st = dict(kind=kind, S=S)
        if kind == "newton":
            st.update(_barrier(g, prob, case["decades"]))
        return st
    if kind == "batch":
        items = []
        for p in range(case["count"]):
            q = _batch_problem(g, case, p)
            b = _barrier(g, q, 1)
            q.update({k: t.cpu().numpy() for k, t in b.items()})
            items.append(q)
        return dict(kind=kind, B=mds.Batch(items, precision=case["precision"]))
    probs = [_batch_problem(g, case, p) for p in range(case["count"])]
    return dict(kind=kind, B=mds.BatchIPM(probs))


# ---- one pass -------------------------------------------------------------
def run(st):
    kind = st["kind"]
    if kind == "newton":
        S = st["S"]
        S.condense(st["sigma_d"], st["dsbase"])
        _, inn, reg = S.factor_inertia(1e-2, reg={})
        steps = 3 if S.precision == "fp64" else 60
        sol, _ = S.refine(st["r_d"], st["r_s"], st["r_y"], steps, 1e-14)
        return dict(dx_d=sol[0], dx_s=sol[1], dy=sol[2], npos=inn["npos"], nzero=inn["nzero"],
                    nneg=inn["nneg"], trials=reg["trials"], delta_w=reg["delta_w"])
    if kind == "ipm":
        r = st["S"].ipm_solve()
        return dict(x=r["x"], y=r["y"], zl=r["zl"], zu=r["zu"], iters=r["iters"], code=r["code"],
                    mu=r["mu"])
    if kind == "batch":
        res = st["B"].run(1e-2)
        return dict(x=torch.cat([t for o in st["B"].out for t in o]),
                    inertia=np.array([r["inertia"] for r in res]),
                    trials=np.array([r["trials"] for r in res]),
                    delta_w=np.array([r["delta_w"] for r in res]))
    if kind == "batch_ipm":
        res = st["B"].solve(trace=False)
        return dict(xy=torch.cat([t for o in st["B"].out for t in o[0][:2]]),
                    iters=np.array([r["iters"] for r in res]),
                    code=np.array([r["code"] for r in res]))
    net = st["net"]
    net.set_params(st["par"])
    loss = [net.train_step(st["X"][k], st["T"][k], 1e-3) for k in range(st["steps"])]
    return dict(params=net.get_params(), pred=net.forward(st["X"][0]), loss=np.array(loss))


# ---- what a pass cannot do without ----------------------------------------
def _newton_work(n_d, n_s, m, r):
    """Read H, J_d, J_s and the vectors once, write the solution once; one
    factorization and one solve."""
    N, nnz = n_d + m, m * r
    return (8.0 * (n_d * n_d + m * n_d + 4 * n_s + 4 * N) + 12.0 * nnz,
            N ** 3 / 3.0 + 2.0 * N * N)


# interior-point iterations that a solve of these problems takes at least
IPM_ITERS = 10


def work(case):
    kind = case["kind"]
    if kind == "mlp_train":
        i, h, o = case["n_in"], case["hidden"], case["n_out"]
        par = i * h + h * h + h * o + i * o
        s = case["steps"]
        return dict(bytes=4.0 * (2 * par + s * case["batch"] * (i + o)),
                    flops=6.0 * par * case["batch"] * s)
    if kind in ("newton", "ipm"):
        b, f = _newton_work(case["n_d"], case["n_s"], case["m"], case["r"])
        return dict(bytes=b, flops=f * (IPM_ITERS if kind == "ipm" else 1))
    tb = tf = 0.0
    for p in range(case["count"]):
        N = case["n_lo"] + (case["n_hi"] - case["n_lo"]) * p // max(case["count"] - 1, 1)
        b, f = _newton_work(N // 4, 50 * N, N - N // 4, 4)
        tb, tf = tb + b, tf + f * (IPM_ITERS if kind == "batch_ipm" else 1)
    return dict(bytes=tb, flops=tf)


# ---- reference in 64 bits --------------------------------------------------
def _exact_newton(prob, st, dev=DEV):
    """Solution of the Newton system by plain torch in FP64: the shifts of the
    correction loop (0, 1e-4, x 100, ...) until both Schur factors are
    definite, then an LU solve of the condensed matrix, refined on the full
    system."""
    nd, ns, m = prob["n_d"], prob["n_s"], prob["m"]
    t = {k: torch.as_tensor(np.ascontiguousarray(prob[k]), device=dev) for k in ("H", "Jd", "v")}
    t.update({k: v.to(dev) for k, v in st.items()})
    r = len(prob["v"]) // m
    row = torch.arange(m, device=dev).repeat_interleave(r)
    col = torch.as_tensor(prob["ci"], device=dev).long()
    order = torch.argsort(col, stable=True)
    row, col, val = row[order], col[order], t["v"][order]
    ptr = torch.searchsorted(col, torch.arange(ns + 1, device=dev))
    cnt = ptr[1:] - ptr[:-1]
    # entries of J_s D^-1 J_s': all pairs within one column
    deg = cnt[col]
    left = torch.arange(len(col), device=dev).repeat_interleave(deg)
    k = torch.arange(len(left), device=dev) - (torch.cumsum(deg, 0) - deg).repeat_interleave(deg)
    right = ptr[col[left]] + k
    eye_d = torch.eye(nd, device=dev, dtype=torch.float64)
    dw, trials = 0.0, 1
    while True:
        Ds = t["dsbase"] + dw
        C = torch.zeros(m, m, device=dev, dtype=torch.float64)
        C.index_put_((row[left], row[right]), val[left] * val[right] / Ds[col[left]],
                     accumulate=True)
        A = t["H"] + torch.diag(t["sigma_d"]) + dw * eye_d
        Lc, bad = torch.linalg.cholesky_ex(C)
        Y = torch.linalg.solve_triangular(Lc, t["Jd"], upper=False)
        _, bad2 = torch.linalg.cholesky_ex(A + Y.T @ Y)
        if int(bad) == 0 and int(bad2) == 0:
            break
        if trials > 12 or int(bad) != 0:
            return None
        dw = 1e-4 if dw == 0.0 else 100.0 * dw
        trials += 1
    M = torch.cat([torch.cat([A, t["Jd"].T], 1), torch.cat([t["Jd"], -C], 1)], 0)
    LU = torch.linalg.lu_factor(M)

    def js(x):
        return torch.zeros(m, device=dev, dtype=torch.float64).index_add_(0, row, val * x[col])

    def jst(y):
        return torch.zeros(ns, device=dev, dtype=torch.float64).index_add_(0, col, val * y[row])

    def solve(rd, rs, ry):
        z = torch.linalg.lu_solve(*LU, torch.cat([rd, ry - js(rs / Ds)])[:, None])[:, 0]
        return z[:nd], (rs - jst(z[nd:])) / Ds, z[nd:]

    rd, rs, ry = t["r_d"], t["r_s"], t["r_y"]
    x = solve(rd, rs, ry)
    for _ in range(2):
        e = solve(rd - A @ x[0] - t["Jd"].T @ x[2], rs - Ds * x[1] - jst(x[2]),
                  ry - t["Jd"] @ x[0] - js(x[1]))
        x = tuple(a + b for a, b in zip(x, e))
    return dict(dx_d=x[0], dx_s=x[1], dy=x[2], npos=nd, nzero=0, nneg=m, trials=trials,
                delta_w=dw)


def exact(case, seed):
    kind = case["kind"]
    if kind == "newton":
        if case["n_d"] + case["m"] > 10000:
            return None  # the reference factorization takes too long there
        g = _gen(seed)
        prob = _problem(g, case["n_d"], case["n_s"], case["m"], case["r"])
        return _exact_newton(prob, _barrier(g, prob, case["decades"]))
    if kind == "batch":
        g, out = _gen(seed), []
        if case["count"] * case["n_hi"] ** 3 > 3e11:
            return None  # hundreds of reference factorizations
        for p in range(case["count"]):
            q = _batch_problem(g, case, p)
            e = _exact_newton(q, _barrier(g, q, 1))
            if e is None:
                return None
            out.append(e)
        return dict(x=torch.cat([e[k] for e in out for k in ("dx_d", "dx_s", "dy")]),
                    inertia=np.array([[e["npos"], 0, e["nneg"]] for e in out]),
                    trials=np.array([e["trials"] for e in out]),
                    delta_w=np.array([e["delta_w"] for e in out]))
    # an interior-point solve and a training epoch end at points that depend
    # on every rounding before them
    return None
