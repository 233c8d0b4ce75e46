"""Column passes with 1, 2, 4 and 8 columns per transform group, and builds on
1, 2 and 4 streams, as chosen by the size of a launch: the same arithmetic per
column and beam, so the S-matrices are equal bit for bit."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu


# 256^2: 8 transform groups' workgroups per beam and column; 512, 256 and 128
# beams per launch are the least that take 8, 4 and 2 columns per group
@pytest.mark.parametrize("batch", [511, 512, 300, 256, 255, 128, 127, 40])
def test_columns_per_group(batch):
    import torch
    import paper_1706_08563_amd as P
    n, L, S, E0 = 256, 25.0, 3, 300e3
    V = np.random.default_rng(5).uniform(0.0, 60.0, size=(S, n, n)).astype(np.float32)
    Vd = torch.from_numpy(V).cuda()
    g = P.prism_grid_init((L, L, 2.0 * S), 2.0, n)
    try:
        P.prism_set_build_streams(1)
        one = P.prism_smatrix_plan(g, E0, 0.024, 2)
        assert one.n_beams >= 513
        whole = P.prism_build_smatrix(one, Vd)
        got = P.prism_build_smatrix(P.prism_smatrix_plan(g, E0, 0.024, 2, beam_batch=batch), Vd)
    finally:
        P.prism_set_build_streams(0)
    by_size = P.prism_build_smatrix(one, Vd)
    torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int32), whole.view(torch.int32))
    assert torch.equal(by_size.view(torch.int32), whole.view(torch.int32))
    beams = O.beam_set(n, L, one.lambda_, 0.024, 2)[[0, 300, len(whole) - 1]]
    ref = O.build_smatrix(V.astype(np.float64), L, 2.0, one.lambda_, one.sigma, beams)
    got3 = whole[[0, 300, len(whole) - 1]].cpu().numpy()
    assert np.linalg.norm(got3 - ref) / np.linalg.norm(ref) <= 1e-5


# batches that do not divide the probes, more and fewer streams, and a batch of
# one: every probe's output is the one it has alone
@pytest.mark.parametrize("n,probes,batch", [(512, 70, 64), (512, 65, 32), (256, 131, 130), (64, 5, 2), (64, 3, 1)])
def test_multislice_batches(n, probes, batch):
    import torch
    import paper_1706_08563_amd as P
    L, S, E0 = 0.1 * n, 2, 200e3
    V = np.random.default_rng(6).uniform(0.0, 60.0, size=(S, n, n)).astype(np.float32)
    Vd = torch.from_numpy(V).cuda()
    g = P.prism_grid_init((L, L, 2.0 * S), 2.0, n)
    xy = np.random.default_rng(7).uniform(0.0, L, size=(probes, 2))
    got = P.multislice_outputs(g, E0, 0.02, Vd, xy, batch=batch)
    alone = torch.cat([P.multislice_outputs(g, E0, 0.02, Vd, xy[p:p + 1], batch=1) for p in (0, probes // 2, probes - 1)])
    assert torch.equal(got[[0, probes // 2, probes - 1]], alone)
    d = P.prism_smatrix_plan(g, E0, 0.02, 1) if n <= 256 else None
    if d is not None:
        ref = O.multislice_outputs(V.astype(np.float64), L, 2.0, d.lambda_, d.sigma, 0.02, xy[:2])
        assert O.rel_err(got[:2].cpu().numpy(), ref) <= 1e-5
