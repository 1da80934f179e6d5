"""The byte and flop model behind the benchmark's trailing-update roofline
(no GPU), against a count over columns."""
import importlib.util
import os

import pytest

_spec = importlib.util.spec_from_file_location(
    "bench_plan", os.path.join(os.path.dirname(__file__), "..", "bench.py"))
bench = importlib.util.module_from_spec(_spec)
_spec.loader.exec_module(bench)


def _update(N, k, w):
    """One update of the lower trailing triangle from row and column k on:
    bytes of its entries (read, write) and of L and W, 2 w flops an entry."""
    n = max(N - k, 0)
    entries = sum(N - c for c in range(k, N))
    return 16.0 * entries + 16.0 * n * w, 2.0 * w * entries


@pytest.mark.parametrize("N,nb", [(10, 4), (1000, 32), (4607, 64), (771, 32)])
def test_single_updates(N, nb):
    b = f = 0.0
    for k in range(nb, N, nb):
        db, df = _update(N, k, nb)
        b, f = b + db, f + df
    assert bench.trailing_plan(N, nb) == (pytest.approx(b), pytest.approx(f))


@pytest.mark.parametrize("N", [4608, 6000, 9001])
def test_pairs_share_an_update(N):
    nb, b, f, k = 64, 0.0, 0.0, 0
    while N - k >= bench.PAIR_ROWS:
        # the strip of the first panel: its columns over all rows below
        n1 = N - k - nb
        b += 16.0 * bench.STRIP_COLS * n1 + 16.0 * n1 * nb
        f += 2.0 * nb * bench.STRIP_COLS * n1
        db, df = _update(N, k + 2 * nb, 2 * nb)
        b, f = b + db, f + df
        k += 2 * nb
    for k0 in range(k + nb, N, nb):
        db, df = _update(N, k0, nb)
        b, f = b + db, f + df
    assert bench.trailing_plan(N, nb) == (pytest.approx(b), pytest.approx(f))


def test_latency_floor_charges_what_a_step_exchanges():
    # 1600 steps, a quarter past the first test: a block's exchange for 16
    # steps, the candidate column's for each of those
    cls = dict(ms=8.0, launches=50)
    tim = {c: dict(ms=0.0, launches=0) for c in ("panel_tail", "trailing", "near")}
    tim["panel"] = cls
    m = bench.panel_latency_model(tim, 1, 1600, 32, dict(coop_steps=1600, coop_second=400, n2x2=0),
                                  dict(block_exchange_us=1.6, candidate_exchange_us=2.0))
    assert m["coop_model"]["us_per_step"] == pytest.approx(5.0)
    assert m["coop_model"]["exchange_floor_us_per_step"] == pytest.approx(0.1 + 0.5)
