"""Infinite and NaN values of S in the two-stage sum: the windows that hold such a
pixel are not finite, and every other probe's pattern is what it is without them,
bit for bit (no product of a padded operand with them, no neighbour's T)."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["PRISM_FP32", "PRISM_SPLIT_BF16X3"])
def test_non_finite_pixel_stays_in_its_windows(prec):
    import torch
    import paper_1706_08563_amd as P
    n, L, f = 256, 25.0, 2
    d = P.prism_smatrix_plan(P.prism_grid_init((L, L, 2.0), 2.0, n), 200e3, 0.020, f)
    S = torch.from_numpy(W.random_complex((d.n_beams, d.ns, d.ns), np.random.default_rng(3))).cuda()
    y, x = np.meshgrid(np.arange(90) * (L / 90), np.arange(70) * (L / 70) + 0.2, indexing="ij")
    xy = np.stack([x.ravel(), y.ravel()], axis=1)
    plan = P.prism_probe_plan_upload(d, xy)

    def run():
        P.prism_timing_reset()
        P.prism_timing_enable(True)
        try:
            out = P.prism_probe_diffraction(d, S, plan, getattr(P, prec))
            assert P.prism_timing_read(P.TIMING_CLASSES["contract"])[1] >= 2       # both sums ran
        finally:
            P.prism_timing_enable(False)
            P.prism_timing_reset()
        return out
    clean = run()
    # the first and the last beam, and one in a ky row's last part-filled step
    bad = [(0, 5, 9, float("inf")), (d.n_beams - 1, 100, 2, float("nan")), (150, 64, 127, float("-inf"))]
    hit = np.zeros(len(xy), bool)
    for b, py, px, v in bad:
        S[b, py, px] = v
        for p in range(len(xy)):
            cx, cy = (O.window_centre(u, L, n) - d.m_win // 2 for u in xy[p])
            hit[p] |= (py - cy) % d.ns < d.m_win and (px - cx) % d.ns < d.m_win
    assert hit.any() and not hit.all()
    got = run()
    hit = torch.from_numpy(hit).cuda()
    assert torch.equal(got[~hit], clean[~hit])
    assert not torch.isfinite(got[hit]).flatten(1).all(1).any()
