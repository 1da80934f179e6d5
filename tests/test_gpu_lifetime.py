"""Destroying a solver or a perceptron waits for nothing but the object's own
calls: not for work on other streams, and it may happen while the thread
captures a stream.  Objects that come and go in several threads keep their
read-backs apart."""
import threading

import numpy as np
import pytest

import paper_2605_13736_amd as mds
import synth

pytestmark = pytest.mark.gpu


def _make(which):
    if which == "solver":
        S = mds.solver_for(synth.config_problem(synth.IPM_N192))
        S.ipm_solve()
        return S
    net = mds.MLP((128, 64, 64, 193), 16)
    x = net.torch.zeros((16, 128), dtype=net.torch.float32, device="cuda")
    net.train_step(x, net.torch.ones((16, 193), dtype=net.torch.float32, device="cuda"), 1e-3)
    return net


@pytest.mark.parametrize("which", ["solver", "mlp"])
def test_destroy_leaves_other_streams_running(which):
    import torch
    obj = _make(which)
    a = torch.randn(8192, 8192, device="cuda")
    side, done = torch.cuda.Stream(), torch.cuda.Event()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(60):  # about 0.4 s
            b = a @ a
        done.record()
    print(f"[gpu-case] destroy {which} beside a busy stream", flush=True)
    obj.close()
    assert not done.query()
    torch.cuda.synchronize()
    assert torch.isfinite(b).all()


@pytest.mark.parametrize("which", ["solver", "mlp", "mlp_wide"])
def test_destroy_during_a_capture(which):
    import torch
    # 70 000 outputs: loss records past the largest block that is kept
    obj = mds.MLP((4, 8, 8, 70000), 32) if which == "mlp_wide" else _make(which)
    x = torch.zeros(1000, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    print(f"[gpu-case] destroy {which} during a capture", flush=True)
    with torch.cuda.graph(g):
        x += 1.0
        obj.close()
        x *= 2.0
    want = 0.0
    for _ in range(3):
        g.replay()
        want = 2.0 * (want + 1.0)
        torch.cuda.synchronize()
        assert (x == want).all()
        x += 0.5  # eager work between the replays
        want += 0.5


def test_objects_in_threads_keep_their_records():
    prob = synth.config_problem(synth.IPM_N192)
    ref = mds.solver_for(prob).ipm_solve()
    out, bad = {}, []

    def work(t):
        import torch
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for k in range(3):
                    S = mds.solver_for(prob)
                    r = S.ipm_solve()
                    out[t, k] = (r["iters"], r["x"].cpu().numpy())
                    S.close()
        except Exception as e:  # reported by the main thread
            bad.append(e)

    print("[gpu-case] solvers in four threads", flush=True)
    ts = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad
    x = ref["x"].cpu().numpy()
    for it, y in out.values():
        assert it == ref["iters"]
        assert np.array_equal(x, y)
