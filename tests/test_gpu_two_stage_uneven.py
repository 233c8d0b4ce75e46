"""Two-stage probe synthesis of scans whose columns are far from equal: columns of
more than 256 probes (found by search instead of one by one) and of a few, more
than 256 columns over a tile, windows over the periodic edge, against the FP64
oracle on sampled probes.

Tolerance (relative Frobenius error of the 3D output): at most 40 roundings per
stage and axis and the window transform's, an amplitude error of 7 x 2^-24 each,
doubled by the square: 2 x 2 x 7 x 2^-24 = 1.7e-6."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("columns,long_columns,long_probes,spread", [(1, 1, 5000, 25.0), (40, 2, 3000, 25.0), (40, 1, 3000, 0.2),
                                                                   (300, 1, 257, 25.0), (16, 16, 256, 25.0)])
def test_uneven_columns(columns, long_columns, long_probes, spread):
    import torch
    import paper_1706_08563_amd as P
    n, L, f, alpha = 256, 25.0, 2, 0.020
    d = P.prism_smatrix_plan(P.prism_grid_init((L, L, 2.0), 2.0, n), 200e3, alpha, f)
    S = W.random_complex((d.n_beams, d.ns, d.ns), np.random.default_rng(columns))
    rng = np.random.default_rng(long_probes)
    x = rng.uniform(0.0, L, size=columns)
    parts = []
    for k in range(columns):
        count = long_probes if k < long_columns else 12
        y = 24.9 + rng.uniform(0.0, spread if k < long_columns else L, size=count)
        parts.append(np.stack([np.full(count, x[k]), y], axis=1))
    xy = rng.permutation(np.concatenate(parts))
    got = P.prism_probe_outputs(d, torch.from_numpy(S).cuda(), P.prism_probe_plan_upload(d, xy), P.PRISM_FP32).cpu().numpy()
    pick = rng.choice(len(xy), size=24, replace=False)
    ref = O.prism_outputs(S.astype(np.complex128), P.prism_beam_list(d).astype(np.int64), L, n, d.lambda_, f, xy[pick])
    assert O.rel_err(got[pick], ref) <= 1.7e-6


def test_one_crowded_column_does_not_slow_the_others():
    """256 columns of 8 probes and one of 20,000 within an Angstrom: every column
    would get the workgroups of the crowded one, 41 million, so the call takes
    the direct sum, a single launch."""
    import torch
    import paper_1706_08563_amd as P
    n, L, f = 1024, 100.0, 4
    d = P.prism_smatrix_plan(P.prism_grid_init((L, L, 20.0), 2.0, n), 200e3, 0.020, f)
    x, y = np.meshgrid(np.arange(256) * (L / 256), np.arange(8) * (L / 8))
    crowd = np.stack([np.full(20000, 50.1), 50.0 + np.random.default_rng(1).uniform(0.0, 1.0, 20000)], axis=1)
    S = torch.randn((d.n_beams, d.ns, d.ns), dtype=torch.complex64, device="cuda")
    for xy, launches in ((np.stack([x.ravel(), y.ravel()], axis=1), None), (crowd, 2),
                         (np.concatenate([np.stack([x.ravel(), y.ravel()], axis=1), crowd]), 1)):
        plan = P.prism_probe_plan_upload(d, xy)
        P.prism_timing_reset()
        P.prism_timing_enable(True)
        try:
            P.prism_probe_outputs(d, S, plan, P.PRISM_SPLIT_BF16X3)
            got = P.prism_timing_read(P.TIMING_CLASSES["contract"])[1]
        finally:
            P.prism_timing_enable(False)
            P.prism_timing_reset()
        assert launches is None or got == launches
