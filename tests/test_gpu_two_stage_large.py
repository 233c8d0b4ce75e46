"""Two-stage probe synthesis beyond 2^31 bytes between the first and the eighth
ky row of T (2048^2, f = 8, 1789 beams, more than 292 scan columns): against the
same scan cut into halves of its columns, which is the same sums and so the same
bits, and against 64 bits on sampled probes.

Tolerance (relative Frobenius error of intensities): at most 47 roundings per
stage and axis and the window transform's, an amplitude error of 7 x 2^-24 each,
doubled by the square: 2 x 2 x 7 x 2^-24 = 1.7e-6."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu


def test_scan_of_320_columns():
    import torch
    import paper_1706_08563_amd as P
    n, L, f = 2048, 200.0, 8
    d = P.prism_smatrix_plan(P.prism_grid_init((L, L, 20.0), 2.0, n), 200e3, 0.024, f)
    assert d.n_beams == 1789 and d.m_win == 128
    g = torch.Generator(device="cuda").manual_seed(4)
    S = torch.randn((d.n_beams, d.ns, d.ns), dtype=torch.complex64, device="cuda", generator=g)
    nx, ny = 320, 48
    y, x = np.meshgrid(np.arange(ny) * (L / ny) + 0.3, np.arange(nx) * (L / nx), indexing="ij")
    x, y = x.T.ravel(), y.T.ravel()                       # column after column
    xy = np.stack([x, y], axis=1)

    def run(part):
        plan = P.prism_probe_plan_upload(d, part)
        P.prism_timing_reset()
        P.prism_timing_enable(True)
        try:
            out = P.prism_probe_diffraction(d, S, plan, P.PRISM_FP32)
            launches = P.prism_timing_read(P.TIMING_CLASSES["contract"])[1]
        finally:
            P.prism_timing_enable(False)
            P.prism_timing_reset()
        return out, launches
    whole, launches = run(xy)
    assert launches == 4                                  # two sums, two passes over the columns
    cut = nx // 2 * ny
    for part, got in ((xy[:cut], whole[:cut]), (xy[cut:], whole[cut:])):
        half, launches = run(part)
        assert launches == 2
        assert torch.equal(half, got)
        del half
    bl = torch.from_numpy(P.prism_beam_list(d).astype(np.float64)).cuda()
    err = ref = 0.0
    for p in np.random.default_rng(5).choice(len(xy), size=6, replace=False):
        rows, cols = ((torch.arange(128, device="cuda") + O.window_centre(v, L, n) - 64) % d.ns for v in (xy[p, 1], xy[p, 0]))
        c = torch.exp(-2j * np.pi * (bl[:, 0] * xy[p, 0] + bl[:, 1] * xy[p, 1]) / L) / np.sqrt(d.n_beams)
        w = S[:, rows][:, :, cols].to(torch.complex128)
        want = torch.fft.fft2((c[:, None, None] * w).sum(0)).abs() ** 2 / 128.0 ** 4
        err += float((whole[p].double() - want).norm() ** 2)
        ref += float(want.norm() ** 2)
    assert (err / ref) ** 0.5 <= 1.7e-6
