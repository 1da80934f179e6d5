"""Batch problems whose first Bunch-Kaufman test fails on most pivots of the x
block, where at most 512 rows go to the register panel (and back): the inertia
(n_d, 0, m) at the first trial, and solutions whose backward error on the Newton
system is within the rounding of the sums, 64 N eps (the batch does not refine
in FP64)."""
import numpy as np
import pytest

import paper_2605_13736_amd as mds

pytestmark = pytest.mark.gpu


def _item(n, kind, seed):
    """n_d = n, m = n: [[H, J'], [J, 0]] with J of full rank, H small and
    indefinite in the columns that fail; one sparse variable apart."""
    rng = np.random.default_rng(seed)
    H = rng.standard_normal((n, n))
    H = 5e-3 * (H + H.T)
    i = np.arange(n)
    strong = {"weak": i < 0, "head": i >= n // 2, "tail": i < n // 2,
              "stripes": i // 40 % 2 == 1}[kind]
    H[i[strong], i[strong]] += 100.0 * n
    J = rng.standard_normal((n, n))
    return dict(n_d=n, n_s=1, m=n, H=np.asfortranarray(H), Jd=np.asfortranarray(J),
                rp=np.zeros(n + 1, dtype=np.int32), ci=np.zeros(0, dtype=np.int32),
                v=np.zeros(0), sigma_d=np.zeros(n), dsbase=np.full(1, 2.0),
                r_d=rng.standard_normal(n), r_s=np.ones(1), r_y=rng.standard_normal(n))


SIZES = (8, 16, 17, 33, 50, 100, 128, 200, 255, 256, 257, 300, 350)


@pytest.mark.parametrize("kind", ["weak", "head", "tail", "stripes"])
def test_batch_weak_pivots(kind):
    items = [_item(n, kind, 100 + n) for n in SIZES]
    print(f"[gpu-case] batch {kind}", flush=True)
    B = mds.Batch(items)
    eps = np.finfo(float).eps
    for _ in range(2):  # the second one replays the graph
        for o in B.out:
            for t in o:
                t.zero_()
        res = B.run(1e-2)
        for it, r, (dx, ds, dy) in zip(items, res, B.out):
            n = it["n_d"]
            assert tuple(r["inertia"]) == (n, 0, n) and r["trials"] == 1
            A = np.block([[it["H"], it["Jd"].T], [it["Jd"], np.zeros((n, n))]])
            x = np.concatenate([dx.cpu().numpy(), dy.cpu().numpy()])
            b = np.concatenate([it["r_d"], it["r_y"]])
            scale = np.abs(A).sum(1).max() * np.abs(x).max() + np.abs(b).max()
            assert np.abs(A @ x - b).max() <= 64 * 2 * n * eps * scale
            assert ds.cpu().numpy()[0] == 0.5


def test_batch_weak_trials():
    # indefinite dense problems: the trials before the shift suffices factor weak
    # matrices, their number and the shift follow from the least eigenvalue
    rng = np.random.default_rng(5)
    items = []
    for n in (40, 101, 300, 512, 513, 700):
        A = rng.standard_normal((n, n))
        A = 0.5 * (A + A.T)
        A[np.arange(n), np.arange(n)] *= 0.01
        it = _item(n, "weak", n)
        it.update(m=0, H=np.asfortranarray(A), Jd=np.zeros((0, n)), rp=np.zeros(1, dtype=np.int32),
                  r_y=np.zeros(0))
        items.append(it)
    print("[gpu-case] batch of indefinite dense problems", flush=True)
    B = mds.Batch(items)
    for it, r, (dx, _, _) in zip(items, B.run(1e-2), B.out):
        n, lo = it["n_d"], np.linalg.eigvalsh(it["H"]).min()
        dw, trials = 1e-4, 2
        while lo + dw <= 0.0:
            dw, trials = 100.0 * dw, trials + 1
        assert tuple(r["inertia"]) == (n, 0, 0)
        assert r["trials"] == trials and r["delta_w"] == pytest.approx(dw, rel=1e-14)
        A = it["H"] + dw * np.eye(n)
        x = dx.cpu().numpy()
        eps = np.finfo(float).eps
        scale = np.abs(A).sum(1).max() * np.abs(x).max() + np.abs(it["r_d"]).max()
        assert np.abs(A @ x - it["r_d"]).max() <= 64 * n * eps * scale
