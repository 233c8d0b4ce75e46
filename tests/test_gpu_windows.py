"""Window transforms of every length that stays in LDS: whole diffraction
patterns and binned outputs, one probe and more probes than the GPU has compute
units, against the FP64 oracle on sampled probes.

Tolerance (relative Frobenius error of intensities): FP32 sums of at most 40
roundings and two transforms of at most 7 radix-2 steps, an amplitude error of
2 x 7 x 2^-24, doubled by the square: 1.7e-6."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

TOL = 1.7e-6


@pytest.mark.parametrize("n_probes", [1, 517])
@pytest.mark.parametrize("n,L,f,alpha,m", [(128, 25.0, 4, 0.012, 16), (128, 20.0, 2, 0.012, 32),
                                           (256, 20.0, 2, 0.012, 64), (256, 20.0, 1, 0.012, 128)])
def test_windows_4d_and_bins(n, L, f, alpha, m, n_probes):
    import torch
    import paper_1706_08563_amd as P
    d = P.prism_smatrix_plan(P.prism_grid_init((L, L, 2.0), 2.0, n), 200e3, alpha, f)
    assert d.m_win == m
    rng = np.random.default_rng(m + n_probes)
    S = W.random_complex((d.n_beams, d.ns, d.ns), rng)
    Sd = torch.from_numpy(S).cuda()
    xy = rng.uniform(-L, 2.0 * L, size=(n_probes, 2))
    plan = P.prism_probe_plan_upload(d, xy, C1=30.0)
    pat = P.prism_probe_diffraction(d, Sd, plan, P.PRISM_FP32).cpu().numpy()
    out = P.prism_probe_outputs(d, Sd, plan, P.PRISM_FP32).cpu().numpy()
    pick = rng.choice(n_probes, size=min(n_probes, 12), replace=False)
    bl = P.prism_beam_list(d).astype(np.int64)
    S64 = S.astype(np.complex128)
    assert O.rel_err(pat[pick], O.prism_diffraction(S64, bl, L, n, d.lambda_, f, xy[pick], C1=30.0)) <= TOL
    assert O.rel_err(out[pick], O.prism_outputs(S64, bl, L, n, d.lambda_, f, xy[pick], C1=30.0)) <= TOL
