"""The perceptron's fused launches at the edges of their tiles.

One training step and one inference call for widths of 1, one entry past a
32-wide tile, sums past a batch of 64 loads, and products large enough for
64 x 64 tiles (128 of them or more), against the FP64 reference on the same
FP32 parameters.

Bars: an output is a sum of K products in FP32 (K <= 1100 + 600 here), so its
error is at most K 2^-24 = 1e-4 of sum |a b|, and for independent signs about
sqrt(K) 2^-24 of max |Y|: 1e-4 relative to max |Y|.  A gradient sums over the
batch what two such layers made: 1e-3 relative to its largest entry, the loss
1e-5.  The Adam step is compared from the gradient read back, as the update of
one entry: 1e-6 at a rate of 1e-3; the second step from the first one's moments.
"""
import numpy as np
import pytest

import paper_2605_13736_amd as mds
from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,batch,max_batch", [
    ((1, 1, 1, 1), 1, 1),
    ((3, 5, 7, 2), 2, 9),
    ((33, 65, 65, 31), 33, 33),
    ((70, 32, 32, 257), 1, 1),
    ((64, 96, 96, 64), 64, 128),
    ((65, 129, 129, 66), 17, 40),
    ((600, 530, 530, 1100), 97, 97),
])
def test_mlp_step_shapes(dims, batch, max_batch):
    print(f"[gpu-case] mlp {dims} batch {batch}", flush=True)
    rng = np.random.default_rng(sum(dims) + batch)
    p = (omlp.init_params(dims, 3) + 0.02 * rng.standard_normal(omlp.n_params(dims)))
    p = p.astype(np.float32).astype(np.float64)
    X = rng.standard_normal((batch, dims[0])).astype(np.float32).astype(np.float64)
    T = rng.standard_normal((batch, dims[3])).astype(np.float32).astype(np.float64)
    net = mds.MLP(dims, max_batch)
    net.set_params(p.astype(np.float32))
    Yr, _ = omlp.forward(p, dims, X)
    for prec, tol in (("fp32", 1e-4), ("bf16", 3e-2)):
        Y = net.forward(X, precision=prec).cpu().numpy().astype(np.float64)
        assert np.abs(Y - Yr).max() <= tol * np.abs(Yr).max(), prec
    m = v = np.zeros_like(p)
    for step in (1, 2):
        loss = net.train_step(X, T, 1e-3)
        g = net.get_grad().astype(np.float64)
        Lr, gr = omlp.loss_and_grad(p, dims, X, T)
        assert loss == pytest.approx(Lr, rel=1e-5), step
        assert np.abs(g - gr).max() <= 1e-3 * np.abs(gr).max(), step
        p1 = net.get_params().astype(np.float64)
        pr, m, v = omlp.adam_step(p, g, m, v, step, 1e-3)
        assert np.abs(p1 - pr).max() <= 1e-6, step
        p = p1
