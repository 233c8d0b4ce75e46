"""Probe synthesis in two stages (sums over kx per scan column, then over ky):
scans of every window size, in any order of the probes, with columns of unequal
length, aberrations, positions outside the cell, and more columns than the
scratch holds at once, against the FP64 oracle on sampled probes.

Tolerances (relative Frobenius error of the 3D output): FP32, at most 40
roundings per stage and axis and the window transform's, an amplitude error of
7 x 2^-24 each: 2 x 2 x 7 x 2^-24 = 1.7e-6; split, the S-matrix rounded at
2^-17, random over beams and pixels: 2 x 2^-17."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

TOL = {"PRISM_FP32": 1.7e-6, "PRISM_SPLIT_BF16X3": 2.0 ** -16}


def _scan(L, nx, ny, seed, order, drop):
    rng = np.random.default_rng(seed)
    x, y = (np.arange(k) * (L / k) + rng.uniform(0.0, 2.0 * L) - L for k in (nx, ny))
    xy = np.stack([g.ravel() for g in np.meshgrid(x, y)], axis=1)
    if order == "columns":
        xy = xy.reshape(ny, nx, 2).transpose(1, 0, 2).reshape(-1, 2)
    if order == "shuffled":
        xy = rng.permutation(xy)
    if drop:
        xy = xy[rng.random(len(xy)) > drop]
    return np.ascontiguousarray(xy)


@pytest.mark.parametrize("prec", sorted(TOL))
@pytest.mark.parametrize("n,L,f,alpha,nx,ny,order,drop,C1",
                         [(256, 25.0, 2, 0.020, 128, 128, "rows", 0.0, 0.0),       # four passes over the columns
                          (256, 25.0, 2, 0.020, 37, 171, "shuffled", 0.3, 80.0),   # more than 64 probes over a tile
                          (256, 25.0, 2, 0.020, 150, 41, "columns", 0.1, 0.0),     # more than 64 columns over a tile
                          (128, 25.0, 4, 0.012, 300, 300, "rows", 0.0, -40.0),     # 16^2 windows
                          (128, 20.0, 2, 0.012, 200, 150, "shuffled", 0.2, 0.0),   # 32^2 windows
                          (256, 20.0, 1, 0.012, 60, 50, "rows", 0.0, 0.0),         # windows of the whole grid, 128^2
                          (512, 40.0, 1, 0.008, 40, 44, "rows", 0.1, 0.0)])        # 256^2 windows
def test_two_stage_scans(prec, n, L, f, alpha, nx, ny, order, drop, C1):
    import torch
    import paper_1706_08563_amd as P
    d = P.prism_smatrix_plan(P.prism_grid_init((L, L, 2.0), 2.0, n), 200e3, alpha, f)
    S = W.random_complex((d.n_beams, d.ns, d.ns), np.random.default_rng(n + f))
    xy = _scan(L, nx, ny, nx, order, drop)
    plan = P.prism_probe_plan_upload(d, xy, C1=C1)
    P.prism_timing_reset()
    P.prism_timing_enable(True)
    try:
        got = P.prism_probe_outputs(d, torch.from_numpy(S).cuda(), plan, getattr(P, prec)).cpu().numpy()
        launches = P.prism_timing_read(P.TIMING_CLASSES["contract"])[1]
    finally:
        P.prism_timing_enable(False)
        P.prism_timing_reset()
    # both sums ran (the one-stage sum is one launch, which the split of the
    # smallest windows still takes)
    assert launches >= 2 or (prec != "PRISM_FP32" and d.m_win == 16)
    pick = np.random.default_rng(1).choice(len(xy), size=24, replace=False)
    bl = P.prism_beam_list(d).astype(np.int64)
    ref = O.prism_outputs(S.astype(np.complex128), bl, L, n, d.lambda_, f, xy[pick], C1=C1)
    assert O.rel_err(got[pick], ref) <= TOL[prec]


def test_two_stage_equals_one_stage_and_keeps_other_probes():
    """The same scan with every x its own value (one stage), and the same
    scan cut in two plans."""
    import torch
    import paper_1706_08563_amd as P
    n, L = 256, 25.0
    d = P.prism_smatrix_plan(P.prism_grid_init((L, L, 2.0), 2.0, n), 200e3, 0.020, 2)
    S = torch.from_numpy(W.random_complex((d.n_beams, d.ns, d.ns), np.random.default_rng(2))).cuda()
    xy = _scan(L, 100, 100, 5, "rows", 0.0)
    whole = P.prism_probe_outputs(d, S, P.prism_probe_plan_upload(d, xy))
    jitter = xy.copy()
    jitter[:, 0] += np.arange(len(xy)) * 1e-13
    one = P.prism_probe_outputs(d, S, P.prism_probe_plan_upload(d, jitter))
    assert float((whole - one).norm() / one.norm()) <= TOL["PRISM_FP32"]
    halves = [P.prism_probe_outputs(d, S, P.prism_probe_plan_upload(d, part)) for part in (xy[:5000], xy[5000:])]
    assert float((torch.cat(halves) - whole).norm() / whole.norm()) <= TOL["PRISM_FP32"]
    # repeats bit for bit, alone and beside another request
    jobs = [(d, S, P.prism_probe_plan_upload(d, part), torch.empty_like(h)) for part, h in zip((xy[:5000], xy[5000:]), halves)]
    for a, b in zip(P.prism_probe_outputs_batched(jobs), halves):
        assert torch.equal(a, b)
