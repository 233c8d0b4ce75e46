"""The rule between the one-stage and the two-stage probe sum (synth_route.hpp,
compiled here by the host compiler) on calls measured on both routes, given by
the sizes that their plans have: where one route takes well over the other's
time, the rule takes the faster one."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1706_08563_amd", "csrc")

SHIM = """
#include "launch_limits.hpp"
#include "synth_route.hpp"
extern "C" int two_stages(int fp32, long probes, long beams, long entries, long tiles, long per_tile, long cols, long rows,
                          long ns, long m, long max_cols, long max_probes, long scratch, double s_bytes) {
    const long step = prism::two_stage_columns_per_launch(cols, rows, ns, m, scratch);
    const long kx = prism::sum_kx_tiles(ns, max_cols);
    const long blocks = kx * prism::sum_kx_row_groups(kx, rows, 3, 256) + prism::sum_ky_blocks(step, ns, m, max_probes);
    return prism::two_stage_route({(bool)fp32, probes, beams, entries, tiles, per_tile, cols, (cols + step - 1) / step, rows,
                                   ns, m, max_probes, blocks, s_bytes});
}
extern "C" int records(long entries, long exact, long tiles, long beams, long ns) {
    return prism::bf16_records_route(entries, exact, tiles, beams, ns);
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("route")
    src, so = d / "shim.cpp", d / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC, str(src), "-o", str(so)], check=True)
    lib = ctypes.CDLL(str(so))
    f, lib.records.argtypes = lib.two_stages, [ctypes.c_long] * 5
    f.records = lib.records
    f.argtypes = [ctypes.c_int] + [ctypes.c_long] * 12 + [ctypes.c_double]
    return f


def _most_in_run(corners, length, ns):
    c = np.bincount(corners, minlength=ns)
    w = np.concatenate([c, c])
    s = np.concatenate([[0], np.cumsum(w)])
    length = min(length, ns)
    return int((s[length:length + ns] - s[:ns]).max())


# (n, L, alpha, f, columns, probes per column), microseconds of one and of two
# stages in FP32 and split BF16 (None: near enough for either)
CALLS = [
    ((256, 25.0, 0.020, 2, 128, 128), (1573, 580), (915, 570)),
    ((256, 25.0, 0.020, 2, 16, 16), (54, 57), (41, 54)),
    ((256, 25.0, 0.020, 2, 256, 16), None, (238, 469)),
    ((256, 25.0, 0.020, 2, 512, 16), (551, 1042), (340, 991)),
    ((256, 25.0, 0.020, 2, 1000, 16), (1080, 2512), None),
    ((256, 25.0, 0.020, 2, 400, 32), None, (616, 896)),
    ((512, 50.0, 0.020, 4, 128, 128), (1591, 650), (924, 622)),
    ((512, 50.0, 0.020, 4, 20, 20), (84, 130), (62, 122)),
    ((512, 50.0, 0.020, 4, 512, 16), (819, 1612), (478, 1574)),
    ((512, 50.0, 0.020, 2, 128, 128), (14306, 2320), (7561, 2271)),
    ((512, 50.0, 0.020, 2, 12, 12), None, (190, 264)),
    ((512, 50.0, 0.020, 2, 256, 16), None, (1879, 2756)),
    ((512, 50.0, 0.020, 2, 512, 16), None, (3758, 5957)),
    ((512, 50.0, 0.020, 2, 1024, 8), (7122, 11598), (3736, 11525)),
    ((1024, 100.0, 0.020, 4, 128, 128), (14518, 3191), (7741, 3032)),
    ((1024, 100.0, 0.020, 4, 16, 16), (663, 894), (540, 815)),
    ((1024, 100.0, 0.020, 4, 512, 16), None, (5133, 9410)),
    ((1024, 100.0, 0.020, 4, 1024, 8), (9466, 20750), (4962, 20712)),
    ((2048, 200.0, 0.020, 8, 256, 256), (61986, 13197), (32451, 12437)),
]


@pytest.mark.parametrize("call,fp32,split", CALLS)
def test_faster_route_is_taken(rule, call, fp32, split):
    import paper_1706_08563_amd as P
    n, L, alpha, f, nx, ny = call
    d = P.prism_smatrix_plan(P.prism_grid_init((L, L, 20.0), 2.0, n), 200e3, alpha, f)
    x, y = np.arange(nx) * (L / nx) + 0.37, np.arange(ny) * (L / ny) + 0.11
    yy, xx = np.meshgrid(y, x, indexing="ij")
    plan = P.prism_probe_plan_init(d, np.stack([xx.ravel(), yy.ravel()], axis=1))
    cx, cy = (np.floor(v * d.ns / L).astype(np.int64) % d.ns for v in (x, y))
    ns, m, rows = d.ns, d.m_win, len(np.unique(P.prism_beam_list(d)[:, 1]))
    for times, is_fp32 in ((fp32, 1), (split, 0)):
        if times is None:
            continue
        one, two = times
        got = rule(is_fp32, nx * ny, d.n_beams, plan.n_entries, plan.n_tiles, plan.max_per_tile, nx, rows, ns, m,
                   _most_in_run(cx, m + 15, ns), _most_in_run(cy, m + 128 // min(m, 128) - 1, ns),
                   (d.n_beams + 15) // 16 * 16 * ns * ns * 8, float(d.smatrix_bytes))
        assert bool(got) == (two < one), (call, times)


def test_one_crowded_column_takes_one_stage(rule):
    """256 columns of 8 probes and one of 20,000 (n = 1024, f = 4, 1245 beams)."""
    common = (1245, 1430000, 70000, 20008)
    assert not rule(0, 22048, *common, 257, 39, 512, 128, 80, 20008, 1248 * 512 * 512 * 8, 1245 * 512 * 512 * 8.0)


# (n, L, alpha, f, probes along each axis), microseconds in plain BF16 from S and with its records
BF16 = [
    ((1024, 100.0, 0.020, 4, 256), (21822, 15528)), ((1024, 100.0, 0.020, 4, 128), (5813, 4435)),
    ((1024, 100.0, 0.020, 4, 64), (1806, 1648)), ((1024, 100.0, 0.020, 4, 32), (733, 1026)),
    ((2048, 200.0, 0.020, 8, 256), (24693, 17863)), ((2048, 200.0, 0.020, 8, 64), (3084, 4112)),
    ((512, 50.0, 0.020, 2, 64), (1457, 1098)), ((512, 50.0, 0.020, 2, 20), (278, 377)),
    ((1024, 100.0, 0.010, 2, 64), (7235, 5981)), ((256, 25.0, 0.020, 2, 16), (35, 46)),
    ((64, 10.0, 0.024, 2, 64), (31, 34)),
]


@pytest.mark.parametrize("call,times", BF16)
def test_bf16_records_where_they_pay(rule, call, times):
    import paper_1706_08563_amd as P
    n, L, alpha, f, k = call
    d = P.prism_smatrix_plan(P.prism_grid_init((L, L, 20.0), 2.0, n), 200e3, alpha, f)
    x = np.arange(k) * (L / k)
    yy, xx = np.meshgrid(x + 0.11, x + 0.37, indexing="ij")
    p = P.prism_probe_plan_init(d, np.stack([xx.ravel(), yy.ravel()], axis=1))
    got = rule.records(p.n_entries, k * k * (d.m_win // 16) ** 2, p.n_tiles, d.n_beams, d.ns)
    assert bool(got) == (times[1] < times[0])
