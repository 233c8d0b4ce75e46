"""The beam contraction at the edges of its tiles: beam counts around the
8-beam step and the 16-beam K step, probe counts around the 32-probe row block
and the 64-probe workgroup, against the FP64 oracle.

Tolerances (relative Frobenius error of the 4D output; an intensity carries
twice the relative error of its amplitude):
  FP32   three BF16 parts leave 2^-25 per product; about 100 FP32 roundings
         (sums and window transform) add 10 x 2^-24: 2 x 10 x 2^-24 = 1.2e-6
  split  parts round at 2^-17 each and lo x lo (2^-16) is left out: 2 x 2^-16
  BF16   operands round at 2^-9 each: 2 x 2^-8
"""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

TOL = {"PRISM_FP32": 1.2e-6, "PRISM_SPLIT_BF16X3": 2.0 ** -15, "PRISM_BF16": 2.0 ** -7}
N, L, E0, F = 64, 10.0, 200e3, 2


@pytest.fixture(scope="module")
def P():
    import torch
    import paper_1706_08563_amd as P
    assert torch.cuda.is_available()
    return P


def _setup(P, alpha, seed):
    import torch
    d = P.prism_smatrix_plan(P.prism_grid_init((L, L, 2.0), 2.0, N), E0, alpha, F)
    S = W.random_complex((d.n_beams, d.ns, d.ns), np.random.default_rng(seed))
    return d, S, torch.from_numpy(S).cuda()


@pytest.mark.parametrize("prec", sorted(TOL))
@pytest.mark.parametrize("alpha,beams,probes", [(0.002, 1, 1), (0.006, 5, 31), (0.0085, 9, 32), (0.0125, 21, 33),
                                                (0.016, 37, 64), (0.024, 69, 65), (0.024, 69, 200)])
def test_contraction_edges(P, prec, alpha, beams, probes):
    d, S, Sd = _setup(P, alpha, 100 + probes)
    bl = P.prism_beam_list(d)
    assert d.n_beams == beams == len(bl)
    # positions within one pixel of each other: their windows share every tile
    xy = 3.0 + np.random.default_rng(probes).uniform(0.0, 0.3, size=(probes, 2))
    xy[::5] += 4.0
    got = P.prism_probe_diffraction(d, Sd, P.prism_probe_plan_upload(d, xy), getattr(P, prec)).cpu().numpy()
    ref = O.prism_diffraction(S.astype(np.complex128), bl.astype(np.int64), L, N, d.lambda_, F, xy)
    assert O.rel_err(got, ref) <= TOL[prec]


@pytest.mark.parametrize("prec", sorted(TOL))
def test_non_finite_pixel_stays_in_its_windows(P, prec):
    import torch
    d, S, Sd = _setup(P, 0.024, 7)
    rng = np.random.default_rng(8)
    xy = rng.uniform(0.0, L, size=(90, 2))
    plan = P.prism_probe_plan_upload(d, xy)
    clean = P.prism_probe_diffraction(d, Sd, plan, getattr(P, prec))
    Sd[20, 5, 9] = float("inf")
    Sd[33, 30, 2] = float("nan")
    got = P.prism_probe_diffraction(d, Sd, plan, getattr(P, prec))
    hit = np.zeros(len(xy), bool)
    for p, (x, y) in enumerate(xy):
        cx, cy = (O.window_centre(v, L, N) - d.m_win // 2 for v in (x, y))
        for py, px in ((5, 9), (30, 2)):
            hit[p] |= (py - cy) % d.ns < d.m_win and (px - cx) % d.ns < d.m_win
    assert hit.any() and not hit.all()
    hit = torch.from_numpy(hit).cuda()
    assert torch.equal(got[~hit], clean[~hit])
    assert not torch.isfinite(got[hit]).flatten(1).all(1).any()


@pytest.mark.parametrize("prec", sorted(TOL))
def test_large_launch_repeats_small_ones(P, prec):
    """Twelve jobs of about 96 workgroups in one launch (two column blocks per
    wave) against each alone (one): the same sums in the same order."""
    import torch
    d, S, Sd = _setup(P, 0.024, 9)
    rng = np.random.default_rng(10)
    plans = [P.prism_probe_plan_upload(d, rng.uniform(0.0, L, size=(1500, 2))) for _ in range(12)]
    alone = [P.prism_probe_outputs(d, Sd, plan, getattr(P, prec)) for plan in plans]
    jobs = [(d, Sd, plan, torch.empty_like(a)) for plan, a in zip(plans, alone)]
    for got, a in zip(P.prism_probe_outputs_batched(jobs, getattr(P, prec)), alone):
        assert torch.equal(got, a)
