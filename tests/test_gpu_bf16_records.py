"""Plain BF16 calls that convert the S-matrix to records first: the same sums as
from S itself, bit for bit, so a large call equals its parts, which are small
enough to read S; beam counts that do not fill the last step of 8 and of 16,
beam chunks, several jobs on one S-matrix.  Against the FP64 oracle on sampled
probes.

Tolerance (relative Frobenius error of intensities): operands round at 2^-9 each:
2 x 2^-8."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu
L = 25.0


def _timed(P, fn):
    P.prism_timing_reset()
    P.prism_timing_enable(True)
    try:
        out = fn()
        return out, P.prism_timing_read(P.TIMING_CLASSES["split"])[1]
    finally:
        P.prism_timing_enable(False)
        P.prism_timing_reset()


# 305 and 293 beams: 1 and 5 past the last K step; windows of 64^2, 128^2 and 32^2
@pytest.mark.parametrize("n,f,alpha,probes", [(256, 2, 0.020, 6000), (256, 1, 0.010, 1500), (256, 4, 0.020, 60000)])
def test_records_repeat_the_direct_sum(n, f, alpha, probes):
    import torch
    import paper_1706_08563_amd as P
    d = P.prism_smatrix_plan(P.prism_grid_init((L, L, 2.0), 2.0, n), 200e3, alpha, f)
    rng = np.random.default_rng(probes)
    S = W.random_complex((d.n_beams, d.ns, d.ns), rng)
    Sd = torch.from_numpy(S).cuda()
    xy = rng.uniform(0.0, L, size=(probes, 2))
    plan = P.prism_probe_plan_upload(d, xy)
    whole, converted = _timed(P, lambda: P.prism_probe_outputs(d, Sd, plan, P.PRISM_BF16))
    assert converted == 1
    parts = np.array_split(np.arange(probes), 40)
    for k in (0, 17, 39):
        few, converted = _timed(P, lambda: P.prism_probe_outputs(d, Sd, P.prism_probe_plan_upload(d, xy[parts[k]]), P.PRISM_BF16))
        assert converted == 0
        assert torch.equal(few, whole[torch.from_numpy(parts[k]).cuda()])
    pick = rng.choice(probes, size=12, replace=False)
    ref = O.prism_outputs(S.astype(np.complex128), P.prism_beam_list(d).astype(np.int64), L, n, d.lambda_, f, xy[pick])
    assert O.rel_err(whole[torch.from_numpy(pick).cuda()].cpu().numpy(), ref) <= 2.0 ** -7
    # two jobs on one S-matrix: one conversion for both
    halves = [P.prism_probe_plan_upload(d, xy[:probes // 2]), P.prism_probe_plan_upload(d, xy[probes // 2:])]
    jobs = [(d, Sd, p, torch.empty((p.plan.n_probes, p.plan.n_bins), device="cuda")) for p in halves]
    both, converted = _timed(P, lambda: P.prism_probe_outputs_batched(jobs, P.PRISM_BF16))
    assert converted == 1
    assert torch.equal(torch.cat(both), whole)


def test_records_in_beam_chunks():
    import torch
    import paper_1706_08563_amd as P
    d = P.prism_smatrix_plan(P.prism_grid_init((L, L, 2.0), 2.0, 256), 200e3, 0.020, 2)
    rng = np.random.default_rng(11)
    S = torch.from_numpy(W.random_complex((d.n_beams, d.ns, d.ns), rng)).cuda()
    xy = rng.uniform(0.0, L, size=(20000, 2))
    chunk = 100                                           # chunks of 100, 100, 100 and 5 beams
    whole, converted = _timed(P, lambda: P.prism_probe_outputs_chunked(d, S, P.prism_probe_plan_upload(d, xy), P.PRISM_BF16, chunk))
    assert converted == 3                                 # 5 beams are too few
    few, converted = _timed(P, lambda: P.prism_probe_outputs_chunked(d, S, P.prism_probe_plan_upload(d, xy[-300:]), P.PRISM_BF16, chunk))
    assert converted == 0 and torch.equal(few, whole[-300:])
