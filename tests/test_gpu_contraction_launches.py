"""Launches of the direct sum with one and with two column blocks per wave, which
the number of workgroups decides (1024, in split and plain BF16): the same sums in
the same order, also for several jobs in one launch."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
MIN_BLOCKS = 1024


def _blocks(plan):
    return plan.plan.n_tiles * max(1, -(-plan.plan.max_per_tile // 64))


@pytest.mark.parametrize("prec", ["PRISM_SPLIT_BF16X3", "PRISM_BF16"])
def test_one_and_two_column_blocks(prec):
    import torch
    import paper_1706_08563_amd as P
    n, L = 64, 10.0
    d = P.prism_smatrix_plan(P.prism_grid_init((L, L, 2.0), 2.0, n), 200e3, 0.024, 2)
    S = torch.from_numpy(W.random_complex((d.n_beams, d.ns, d.ns), np.random.default_rng(9))).cuda()
    rng = np.random.default_rng(10)
    plans = [P.prism_probe_plan_upload(d, rng.uniform(0.0, L, size=(1500, 2))) for _ in range(24)]
    assert all(_blocks(p) < MIN_BLOCKS for p in plans) and sum(map(_blocks, plans)) >= MIN_BLOCKS
    alone = [P.prism_probe_outputs(d, S, p, getattr(P, prec)) for p in plans]
    jobs = [(d, S, p, torch.empty_like(a)) for p, a in zip(plans, alone)]
    for got, a in zip(P.prism_probe_outputs_batched(jobs, getattr(P, prec)), alone):
        assert torch.equal(got, a)
    one = P.prism_probe_plan_upload(d, np.concatenate([p.xy for p in plans]))
    assert _blocks(one) >= MIN_BLOCKS
    assert torch.equal(P.prism_probe_outputs(d, S, one, getattr(P, prec)), torch.cat(alone))
