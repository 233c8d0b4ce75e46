"""Host cost of probe plans (no GPU)."""
import time

import numpy as np
import pytest


def _seconds(P, d, xy):
    best = float("inf")
    for _ in range(3):
        t0 = time.perf_counter()
        P.prism_probe_plan_init(d, xy)
        best = min(best, time.perf_counter() - t0)
    return best


@pytest.mark.parametrize("step", [1.0 / 64, 1.0 / 256, 1.0 / 1024])
def test_positions_on_binary_fractions_cost_no_more(step):
    """Positions whose low mantissa bits are zero, each x a value of its own or
    shared by a few probes: the grouping by x takes no longer than for positions
    anywhere (a hash of the low bits took 15 times as long)."""
    import paper_1706_08563_amd as P
    d = P.prism_smatrix_plan(P.prism_grid_init((128.0, 128.0, 20.0), 2.0, 1024), 200e3, 0.010, 4)
    xy = np.random.default_rng(3).uniform(0.0, 128.0, size=(262144, 2))
    assert _seconds(P, d, np.round(xy / step) * step) <= 4.0 * _seconds(P, d, xy)
