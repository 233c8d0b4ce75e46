"""Host arithmetic of the launch sizes (launch_limits.hpp, compiled here by the
host compiler), over every grid, interpolation factor and aperture."""
import ctypes
import itertools
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1706_08563_amd", "csrc")

SHIM = """
#include "launch_limits.hpp"
extern "C" int columns(int n_cols, int n_rows, int ns, int m, size_t T_bytes) {
    return prism::two_stage_columns_per_launch(n_cols, n_rows, ns, m, T_bytes);
}
extern "C" int groups(int n_bins) { return prism::bin_groups(n_bins); }
extern "C" int items(int n_bins) { return prism::bin_items(n_bins); }
extern "C" long kx(int ns, int max_cols, int n_rows, int row_steps, int max_steps) {
    const long tiles = prism::sum_kx_tiles(ns, max_cols);
    return tiles * prism::sum_kx_row_groups(tiles, n_rows, row_steps, max_steps);
}
extern "C" long ky(int n_cols, int ns, int m, int max_probes) { return prism::sum_ky_blocks(n_cols, ns, m, max_probes); }
extern "C" int streams(int n, long items, long batches) { return prism::streams_by_size(n, items, batches); }
extern "C" int launchable(long blocks) { return prism::launchable(blocks); }
"""


@pytest.fixture(scope="module")
def limits(tmp_path_factory):
    d = tmp_path_factory.mktemp("limits")
    src, so = d / "shim.cpp", d / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC, str(src), "-o", str(so)], check=True)
    lib = ctypes.CDLL(str(so))
    lib.columns.argtypes = [ctypes.c_int] * 4 + [ctypes.c_size_t]
    lib.kx.restype = lib.ky.restype = ctypes.c_long
    lib.launchable.argtypes = [ctypes.c_long]
    lib.streams.argtypes = [ctypes.c_int, ctypes.c_long, ctypes.c_long]
    return lib


def _last_offset(n_cols, ns, m):
    """Largest byte offset + 8 of a load of the second sum: value (row of the
    tile, window column) of the eighth ky from a base at its first."""
    w = min(m, 128)
    return 8 * (7 * ns * n_cols * m + (128 // w - 1) * n_cols * m + (m - 1)) + 8


def test_offsets_of_the_second_sum_stay_in_32_bits(limits):
    grids = [(n, f) for n, f in itertools.product((64, 128, 256, 512, 1024, 2048), (1, 2, 4, 8, 16, 32))
             if 16 <= n // 2 // f <= 512]
    for (n, f), n_rows, cols in itertools.product(grids, (1, 9, 40, 64, 257), (1, 2, 64, 147, 255, 256, 293, 320, 4096,
                                                                              (1 << 28) - 1)):
        ns, m = n // 2, n // 2 // f
        for T in (n_rows * ns * m * 8, 1 << 30, 105 << 30):
            if T < n_rows * ns * m * 8:
                continue                                  # a column of T fits, or the call takes the direct sum
            got = limits.columns(cols, n_rows, ns, m, T)
            assert 1 <= got <= cols
            assert got * n_rows * ns * m * 8 <= T
            assert _last_offset(got, ns, m) <= 0x7fffffff
            # and no more launches than these bounds ask for
            assert (got == cols or (got + 1) * n_rows * ns * m * 8 > T
                    or _last_offset(got + 1, ns, m) + 8 * m * (got + 1) > 0x7fffffff)


# 2048^2 at 200 A: (beams, ky rows, f, scan columns) of apertures and
# scans whose T fits the scratch in one launch, and whose offsets do not
@pytest.mark.parametrize("beams,n_rows,f,cols", [(1789, 47, 8, 305), (2925, 61, 8, 320), (4997, 79, 4, 160),
                                                 (4997, 79, 2, 80)])
def test_large_scans_take_more_launches(limits, beams, n_rows, f, cols):
    ns, m = 1024, 1024 // f
    T = (beams + 15) // 16 * 16 * ns * ns * 8
    assert cols * n_rows * ns * m * 8 <= T and _last_offset(cols, ns, m) > 0x7fffffff
    got = limits.columns(cols, n_rows, ns, m, T)
    assert got < cols and _last_offset(got, ns, m) <= 0x7fffffff


def test_bin_sums_hold_fewer_than_2_32_threads(limits):
    for n_bins in (1, 4, 62, 4095, 4096, 4097, 1 << 20, (1 << 22) - 1, 1 << 22, (1 << 22) + 5, 1 << 26, 0x7fffffff):
        g, most = limits.groups(n_bins), limits.items(n_bins)
        assert g >= 1 and most >= 1 and g * most * 256 < 1 << 32
        assert 4 * g >= n_bins or g == 1 << 20              # all bins at once, or 2^22 at a time
    assert limits.items(4096) < 16384                       # 16,384 windows of 4096 bins: two launches


def test_two_stage_launches_hold_fewer_than_2_32_threads(limits):
    assert limits.launchable((1 << 24) - 8) and not limits.launchable((1 << 24) - 7)
    # the benchmark scans, and one column of very many probes beside 256 others
    assert limits.launchable(limits.ky(256, 1024, 128, 256)) and limits.launchable(limits.kx(1024, 256, 39, 3, 256))
    assert not limits.launchable(limits.ky(257, 512, 128, 20000))
    assert not limits.launchable(limits.kx(1024, 65535, 39, 3, 256))
    # a row group's K steps fit its table
    for n_rows in (1, 2, 9, 39, 79, 257):
        for row_steps in (1, 3, 17, 128):
            for tiles in (2, 32, 8192):
                got = _row_groups(limits, tiles, n_rows, row_steps)
                assert 1 <= got <= n_rows
                assert -(-n_rows // got) * row_steps <= 256


def _row_groups(limits, tiles, n_rows, row_steps):
    ns = {2: 16, 32: 64, 8192: 1024}[tiles]
    return limits.kx(ns, 1, n_rows, row_steps, 256) // tiles


# n, items of a batch, batches, times on 1, 2 and 4 streams
@pytest.mark.parametrize("n,items,batches,times", [
    (256, 21, 1, (339, 455, 765)), (256, 69, 1, (308, 310, 472)), (512, 69, 1, (1502, 1374, 1807)),
    (256, 305, 1, (1566, 1408, 1765)), (1024, 1245, 1, (262400, 253900, 249500)),
    (1024, 12, 104, (39700, 37800, 34400)), (1024, 16, 78, (35400, 34900, 32000)), (1024, 20, 63, (37700, 34300, 31500)), (1024, 24, 52, (34400, 31800, 32500)),
    (1024, 31, 41, (32600, 30800, 31300)), (1024, 33, 38, (36970, 30660, 30970)), (1024, 8, 1, (501, 557, 623)),
    (512, 24, 1, (336, 411, 481)), (2048, 40, 1, (219, 231, 236)), (2048, 128, 1, (228, 213, 216)),
    (2048, 256, 1, (248, 224, 217))])
def test_streams_by_size(limits, n, items, batches, times):
    got = limits.streams(n, items, batches)
    assert times[{1: 0, 2: 1, 4: 2}[got]] <= 1.02 * min(times)
