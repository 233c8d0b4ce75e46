"""prism_set_build_streams governs multislice as it does builds: with 1 every
launch runs on the caller's stream, so that their times, which then do not
overlap, add up to no more than the call's; any count gives the same outputs."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_stream_count_of_multislice():
    import torch
    import paper_1706_08563_amd as P
    n, L, slices = 1024, 100.0, 12
    g = P.prism_grid_init((L, L, 2.0 * slices), 2.0, n)
    V = torch.rand((slices, n, n), device="cuda") * 60.0
    xy = np.random.default_rng(1).uniform(0.0, L, size=(128, 2))
    outs, busy = {}, {}
    try:
        for streams in (1, 2, 4, 0):
            P.prism_set_build_streams(streams)
            P.multislice_outputs(g, 200e3, 0.020, V, xy, batch=64)
            torch.cuda.synchronize()
            P.prism_timing_reset()
            P.prism_timing_enable(True)
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            outs[streams] = P.multislice_outputs(g, 200e3, 0.020, V, xy, batch=64)
            b.record()
            torch.cuda.synchronize()
            total = sum(P.prism_timing_read(P.TIMING_CLASSES[k])[0] for k in ("pass_a", "pass_b", "bin_reduce"))
            P.prism_timing_enable(False)
            busy[streams] = total / a.elapsed_time(b)
    finally:
        P.prism_timing_enable(False)
        P.prism_timing_reset()
        P.prism_set_build_streams(0)
    assert busy[1] <= 1.0, busy
    assert busy[2] > 1.2, busy
    for streams in (2, 4, 0):
        assert torch.equal(outs[streams], outs[1])
