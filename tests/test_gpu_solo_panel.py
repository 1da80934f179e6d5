"""The cooperative panel where one workgroup is left (at most 256 rows), and the
search for the largest entry: matrices made of small blocks whose elimination is
exact in FP64 and FP32, so that equal maxima stay equal, at orders around the tile
edges.  The oracle's pivots (the first of equal maxima) and inertia, and the factor
bit for bit the same with every panel and width (in FP64 the memory panel's), with
failing pivots alone and in runs between passing blocks."""
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


def _ties(N, kind):
    """Symmetric: triples of rows [[0, 1, 1], [1, 0, 1], [1, 1, 0]] up to signs,
    scattered over the order; two equal maxima stand in a triple's first column.
    mixed: every other 20 rows have a dominant power of two instead."""
    rng = np.random.default_rng(N)
    rows = np.arange(N)
    A = np.zeros((N, N))
    if kind == "mixed":
        lone = rows // 20 % 2 == 1
        A[rows[lone], rows[lone]] = np.where(rng.random(lone.sum()) < 0.5, 8.0, -8.0)
        rows = rows[~lone]
    rows = rng.permutation(rows)
    for t in range(0, len(rows) - 2, 3):
        for a, b in ((0, 1), (0, 2), (1, 2)):
            i, j = rows[t + a], rows[t + b]
            A[i, j] = A[j, i] = rng.choice((-1.0, 1.0))
    return A  # one or two rows stay zero where the order is no multiple of three


SIZES = [1, 2, 3, 15, 16, 17, 33, 63, 65, 128, 255, 256, 257, 320, 511, 513]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("kind", ["ties", "mixed"])
@pytest.mark.parametrize("N", SIZES)
def test_equal_maxima(N, kind, precision):
    A = _ties(N, kind)
    _, dd, ds, ipo, _, _ = oracle.bk(A)
    io = tuple(oracle.inertia(ipo, dd, ds)[:3])
    out = {}
    for panel, nb in (("mem", 0), ("coop", 0), ("coop", 8), ("coop", 64), ("auto", 0)):
        print(f"[gpu-case] ties N={N} {kind} {precision} panel={panel} nb={nb}", flush=True)
        if panel == "mem" and precision == "fp32":
            continue  # FP64 only
        S = mds.solver_for(_dense_problem(A), panel=panel, nb=nb, precision=precision)
        S.condense(np.zeros(N), np.zeros(0), 0.0, 0.0)
        _, inn, _ = S.factor_inertia()
        L, d, e, piv = S.get_factor()
        assert np.array_equal(piv, ipo), (panel, nb)
        assert (inn["npos"], inn["nzero"], inn["nneg"]) == io, (panel, nb)
        out[panel, nb] = (L, d, e)
        assert S.fallbacks()["coop_aborts"] == 0
        del S
    ref = out["mem" if precision == "fp64" else "coop", 0]  # FP32: of the equilibrated matrix
    for got in out.values():
        for a, b in zip(got, ref):
            assert np.array_equal(a, b)
