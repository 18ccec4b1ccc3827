"""Row lengths around the 128-bit word (four floats), the lanes of a wave and the wide-row threshold: rows that are not
whole words move as 128-bit accesses at any float's address with their last one to three floats on their own, and the
last lane of a column tile overlaps its neighbour.  Every output against the oracle, to the tolerances of the calls'
own tests (floats bit for bit, keys to 1e-12: fp64 sums of at most a few thousand squares in another order)."""
import numpy as np
import pytest

import workloads as wk

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

ROW_LENGTHS = [1, 2, 3, 4, 5, 6, 7, 9, 13, 63, 255, 257, 258, 259, 511, 1023, 2047, 2049, 2050, 2051]


def _workload(mode, R, seed, rows=37):
    shapes = []
    for n in ROW_LENGTHS:
        ci, khw = (n // 3, 3) if n % 3 == 0 else (n, 1)
        G = ci if mode == wk.MODE_CHANNEL else rows
        shape = (rows, ci, khw, mode, max(1, (2 * G) // 5))
        shapes.append(shape + (max(1, ci // 2),) if mode == wk.MODE_BOTH else shape)
    return wk.custom_workload(shapes, R=R, seed=seed, sigma_replica=0.03)


@pytest.mark.parametrize("mode", [wk.MODE_NONE, wk.MODE_FILTER, wk.MODE_CHANNEL, wk.MODE_BOTH])
@pytest.mark.parametrize("R", [1, 4, 5])
def test_row_lengths_that_are_not_whole_words(mode, R):
    from tests.test_gpu_frozen import _check_frozen
    from tests.test_gpu_parity import _run
    from tests.test_gpu_weighted import _phase4_chain
    import oracle
    wl = _workload(mode, R, 10 * R + mode)
    _run(wl, want_wbar=True, want_sqnorm=True)
    W, U = wk.generate(wl)
    rng = np.random.default_rng(77 + R)
    L = len(wl.layers)
    a, b = rng.uniform(0.3, 1.0, L).astype(np.float32), rng.uniform(0.0, 0.7, L).astype(np.float32)
    _phase4_chain(wl, W, U, a, b, rng, fused_dual=True, one_call=True)
    _check_frozen(wl, W, U, oracle.project(wl.table(), W, U)["mask"])


def test_row_lengths_that_are_not_whole_words_with_the_estimate(monkeypatch):
    from tests.test_gpu_parity import _run
    monkeypatch.setenv("HSADMM_FORCE_ESTIMATE", "1")
    _run(_workload(wk.MODE_FILTER, 4, 5), want_wbar=True, want_sqnorm=True)
