"""Bin sums of more (item, bin) wavefronts than one launch holds: 16,384 windows
of 256^2 with a 4096-entry detector map (2^32 threads), against the windows'
whole patterns of sampled probes, and against the same probes in a small call.

Tolerance: a bin's 16 FP32 values in one wavefront's order against a sum in 64
bits, at most 16 roundings of 2^-24: 1e-6."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_more_bins_than_one_launch():
    import torch
    import paper_1706_08563_amd as P
    n, L, f = 1024, 100.0, 2
    d = P.prism_smatrix_plan(P.prism_grid_init((L, L, 20.0), 2.0, n), 200e3, 0.001, f)
    assert d.m_win == 256
    g = torch.Generator(device="cuda").manual_seed(6)
    S = torch.randn((d.n_beams, d.ns, d.ns), dtype=torch.complex64, device="cuda", generator=g)
    xy = np.random.default_rng(7).uniform(0.0, L, size=(16384, 2))
    dmap = np.random.default_rng(8).permutation(256 * 256).reshape(256, 256).astype(np.int32) % 4096
    out = P.prism_probe_outputs(d, S, P.prism_probe_plan_upload(d, xy, n_bins=4096, detector_map=dmap))
    pick = np.array([0, 5000, 16382, 16383])
    few = P.prism_probe_plan_upload(d, xy[pick], n_bins=4096, detector_map=dmap)
    assert torch.equal(P.prism_probe_outputs(d, S, few), out[pick])
    pat = P.prism_probe_diffraction(d, S, few).double().reshape(4, -1)
    idx = torch.from_numpy(dmap.astype(np.int64).ravel()).cuda()
    want = torch.zeros((4, 4096), dtype=torch.float64, device="cuda").index_add_(1, idx, pat)
    assert float(((out[pick].double() - want).abs() / want).max()) <= 1e-6
