// launch_limits.hpp -- how much one launch may hold, and how many streams a call
// takes (plain host C++, no HIP).
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace prism {

// The beam sums read 8 planes (beams, or ky rows of T) from one base address
// with byte offsets that are positive 32-bit integers, and their buffer resource
// ends at 2^31 - 1 bytes: what lies beyond reads as zero.
constexpr int64_t MAX_BUFFER_BYTES = 0x7fffffff;
constexpr int SUM_PLANES = 8;

// Scan columns per launch of the two-stage sum: their T (n_rows ky, ns rows of
// the S grid, m window columns, complex64) fits T_bytes, and the offsets of the
// second sum are in range.  It addresses, from a window row of a scan column,
// the same place 7 planes of ns n m values further, and up to R = 128 / min(m,
// 128) S-grid rows of n m values.  At least 1, which is in range for every ns
// and m up to 2^22 values.  292 columns at ns m = 2^17 (2048^2, f = 8), 73 at
// 2^19.
inline int two_stage_columns_per_launch(int n_cols, int n_rows, int ns, int m, size_t T_bytes) {
    const int64_t value = 8, R = 128 / std::min(m, 128);
    const int64_t reach = MAX_BUFFER_BYTES / (value * m * ((int64_t)(SUM_PLANES - 1) * ns + R));
    const int64_t fit = (int64_t)(T_bytes / ((size_t)n_rows * ns * m * value));
    return (int)std::max<int64_t>(1, std::min<int64_t>({(int64_t)n_cols, fit, reach}));
}

// A launch holds fewer than 2^32 threads.
constexpr int64_t MAX_THREADS = 0xffffffff;
inline int64_t most_blocks(int threads) { return MAX_THREADS / threads; }

// Bin sums, one wavefront per (item, bin): workgroups of 4 bins per item (each
// takes further bins in turn when they are more than 2^22), and items per launch.
inline int bin_groups(int n_bins) { return (int)std::min<int64_t>(((int64_t)n_bins + 3) / 4, 1 << 20); }
inline int bin_items(int n_bins) { return (int)std::min<int64_t>(most_blocks(256) / std::max(1, bin_groups(n_bins)), 1 << 24); }

// Workgroups of the two-stage sum's launches.  First sum: 128-pixel tiles by 64
// scan columns (max_cols over a tile) by row groups, enough for 4096 workgroups
// and at least two per max_steps K steps.  Second sum: 128 window pixels by scan
// columns by 64 probes (max_probes of a column over those pixels).
constexpr int SUM_ROWS = 64;
inline int64_t sum_kx_tiles(int ns, int max_cols) { return (int64_t)ns * ns / 128 * ((max_cols + SUM_ROWS - 1) / SUM_ROWS); }
inline int sum_kx_row_groups(int64_t tiles, int n_rows, int row_steps, int max_steps) {
    const int64_t least = ((int64_t)n_rows * row_steps + max_steps - 1) / max_steps;
    return (int)std::min<int64_t>(n_rows, std::max<int64_t>(2 * least, std::min<int64_t>(4096 / tiles, n_rows)));
}
inline int64_t sum_ky_blocks(int n_cols, int ns, int m, int max_probes) {
    const int w = std::min(m, 128), R = 128 / w;
    return (int64_t)n_cols * (ns / R) * (m / w) * ((max_probes + SUM_ROWS - 1) / SUM_ROWS);
}
// Whether a launch may hold that many workgroups of 256, in 8 equal parts.
inline bool launchable(int64_t blocks) { return (blocks + 7) / 8 * 8 <= most_blocks(256); }

// Streams of a build (or multislice) in batches of `items`.  Each further stream
// costs two launches per slice and shorter kernels; small batches stay on one.
// Builds on 1, 2 and 4 streams:
//   up to 1024^2, by pixels (items x n^2), us
//     21 beams at 256^2 (1.4 M)      339    455    765
//     69 beams at 256^2 (4.5 M)      308    310    472
//     16 probes at 1024^2 (17 M)    3516   3655      -   (multislice, 4 batches)
//     69 beams at 512^2 (18 M)      1502   1374   1807
//     305 beams at 256^2 (20 M)     1566   1408   1765
//     1245 beams at 512^2 (326 M)  23359  22753  23269
//     1245 beams at 1024^2 (1.3 G)  262.4, 253.9 and 249.5 ms
//   many small batches at 1024^2, whose parts run on without waiting for each
//   other: 1245 beams in batches of, ms of 6 slices
//     8     40.3  41.5  37.8
//     12    39.7  37.8  34.4
//     16    35.4  34.9  32.0
//     20    37.7  34.3  31.5
//     24    34.4  31.8  32.5
//     31    32.6  30.8  31.3
//   at 2048^2, by items, us per beam of 10 slices (a batch of 2^k items is the
//   slow one on one stream, and its parts are not)
//     40 beams                     219  231  236
//     64                           219  216  222
//     128                          228  213  216
//     256                          248  224  217
//     305, 1245                    223, 225 within 1%
constexpr int MANY_BATCHES = 8;
inline int streams_by_size(int n, int64_t items, int64_t batches) {
    if (n > 1024) return items < 64 ? 1 : (items < 192 ? 2 : 4);
    const int64_t M = 1 << 20, pixels = items * n * n;
    if (pixels < 8 * M || (items < 32 && batches < MANY_BATCHES)) return 1;
    if (items < 32) return pixels < 24 * M ? 4 : 2;
    return pixels < 700 * M ? 2 : 4;
}

}  // namespace prism
