"""The perceptron's launches of 128 or more 64 x 64 tiles in every kind of piece:
the output layer with its skip product, gradient and loss records (130 tiles),
the hidden layers and their backward product (162), and the first weight's
gradient with Adam behind it (180); FP32 training and FP32 and BF16 inference,
widths and batches that are no multiples of a tile, against the FP64 reference
on the same FP32 parameters.

Bars as for the smaller shapes: sums of at most 1700 FP32 products, so 1e-4 of
max |Y| (3e-2 with BF16 operands), gradients 1e-3 of their largest entry, the
loss 1e-5, the Adam step of an entry 1e-6 at a rate of 1e-3.
"""
import numpy as np
import pytest

import paper_2605_13736_amd as mds
from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


def _tiles(m, n):
    return -(-m // 64) * -(-n // 64)


@pytest.mark.parametrize("dims,batch,big", [
    ((70, 130, 130, 4097), 127, "out"),
    ((600, 1100, 1100, 50), 530, "hidden"),
])
def test_mlp_large_tiles(dims, batch, big):
    print(f"[gpu-case] mlp {dims} batch {batch}", flush=True)
    if big == "out":
        assert _tiles(batch, dims[3]) >= 128
    else:
        assert min(_tiles(batch, dims[1]), _tiles(dims[0], dims[1])) >= 128
    rng = np.random.default_rng(sum(dims) + batch)
    p = (omlp.init_params(dims, 3) + 0.02 * rng.standard_normal(omlp.n_params(dims)))
    p = p.astype(np.float32).astype(np.float64)
    X = rng.standard_normal((batch, dims[0])).astype(np.float32).astype(np.float64)
    T = rng.standard_normal((batch, dims[3])).astype(np.float32).astype(np.float64)
    net = mds.MLP(dims, batch + 3)
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
