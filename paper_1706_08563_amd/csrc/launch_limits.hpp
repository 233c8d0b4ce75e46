// launch_limits.hpp -- how much one launch may hold (plain host C++, no HIP).
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

}  // namespace prism
