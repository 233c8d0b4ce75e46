// synth_route.hpp -- which calls take the two-stage probe sum, and which plain BF16
// calls convert S first (plain host C++).
#pragma once
#include <algorithm>
#include <cstdint>

namespace prism {

struct SynthSizes {
    bool fp32;                                        // FP32, else split BF16
    int64_t n_probes, n_beams, n_entries, n_tiles;    // n_entries: (work tile, probe) pairs
    int64_t max_per_tile;                             // most probes of a work tile
    int64_t n_cols, passes, n_rows, ns, m;            // scan columns, passes over them, ky
    int64_t max_probes;                               // most probes of a column over 128 window pixels
    int64_t blocks;                                   // workgroups of both sums, first pass
    double s_bytes;                                   // S-matrix
    double t_bytes() const { return 8.0 * n_cols * n_rows * ns * m; }
    double window_bytes() const { return 8.0 * n_probes * m * m; }
};

inline int64_t whole(int64_t v, int64_t step) { return (v + step - 1) / step * step; }

// Seconds of the sums (fitted to 560 calls of 64^2 to 2048^2 grids, 16^2 to 512^2
// windows, 25 to 1789 beams, scans of 1 to 1024 columns; 10% at the median).
// One stage: products of whole K steps, with the 16 rows of a row block that a
// tile's last probes leave empty on average; S; workgroups; probes.
inline double one_stage_seconds(const SynthSizes& z) {
    return 20e-6 + (double)(z.n_entries + 16 * z.n_tiles) * 256 * 8 * whole(z.n_beams, 16) / (z.fp32 ? 200e12 : 375e12) +
           z.s_bytes / 25e12 + 32e-9 * (double)(z.n_tiles * ((z.max_per_tile + 63) / 64)) + 0.6e-9 * (double)z.n_probes;
}
// Two: S in every pass, T written and read, windows; the second sum's products,
// padded to 32 probes and 16 ky; passes and workgroups.
inline double two_stage_seconds(const SynthSizes& z) {
    return 8e-6 + 15e-6 * (double)z.passes + (double)z.passes * z.s_bytes / 8.7e12 + z.t_bytes() / 1.6e12 +
           z.window_bytes() / 2.4e12 + 4e-9 * (double)z.blocks +
           (double)(z.n_cols * z.ns * z.m) * whole(z.max_probes, 32) * whole(z.n_rows, 16) * 48 / 1.5e15;
}

// Two stages, when the products they save at least pay for their traffic (S and T,
// and 3 ns for each workgroup: those of a column with few probes are empty beside
// one with many), and when they do not lose by more than the accuracy they bring
// is worth: split BF16 ends 2.3e-7 from 64 bits instead of 6.9e-7, so up to 0.1
// ms or half as long again where a call takes less than that, and otherwise up to
// a third longer, but a tenth where T is more than three times the windows.
// Measured, one and two stages (split BF16 where not said), in us:
//   two     16,384 probes (128 x 128), 305 beams, 64^2 windows at 256^2      915, 570
//           16,384, 1245 beams, 128^2 at 1024^2                             7741, 3032;  FP32 14518, 3191
//           900, 1245 beams, 128^2 at 1024^2, FP32                          1502, 1067
//           8100, 437 beams, 128^2 at 2048^2                                2353, 2730
//   one     256, 305 beams, 64^2 at 256^2                                     41, 54
//           144, 1245 beams, 128^2 at 512^2                                  190, 264
//           8192 (512 columns of 16), 1245 beams, 128^2 at 1024^2           5133, 9410;  FP32 9513, 9576
//           4096 (256 of 16), 1245 beams, 128^2 at 512^2                    1879, 2756;  FP32 3575, 2787
//           16,000 (1000 of 16), 1245 beams, 128^2 at 512^2                 7486, 11630
//           16,000 (1000 of 16), 305 beams, 64^2 at 256^2, FP32             1080, 2512
//           22,048 (256 of 8, one of 20,000), 1245, 128^2 at 1024^2        18200, 127900
inline bool two_stage_route(const SynthSizes& z) {
    const double products = (double)z.n_entries * 256 * 8 * z.n_beams / (z.fp32 ? 130e12 : 230e12);
    const double traffic = 20e-6 + std::max((z.s_bytes + 2 * z.t_bytes()) / 4e12, 3e-9 * (double)z.blocks);
    if (products < 1.15 * traffic) return false;
    const double one = one_stage_seconds(z), part = z.t_bytes() > 3 * z.window_bytes() ? 0.1 : 0.35;
    return two_stage_seconds(z) <= one + std::max(std::min(one / 2, 100e-6), part * one);
}

// Whether plain BF16 converts S to records first (1.5 times S in traffic, then a
// quarter of the load instructions and 3/5 of the cache lines per product): by how
// often each S value is used, and whether the windows fill their work tiles exactly
// (n_entries = exact_entries), as for scans on whole pixels, whose direct sum is
// slowed more by rows of 128 bytes that lie across two lines.  Measured, from S and
// with records, us:
//   uses (products per pixel of S) with full tiles
//       64   1024 probes, 1245 beams at 1024^2        733, 1026
//      256   4096 at 1024^2                          1806, 1648
//     1024   16,384 at 1024^2                        5813, 4435;   65,536 at 2048^2  24693, 17863
//     4096   16,384 at 512^2                         5073, 3743
//   with part-filled tiles
//      281   3600 anywhere at 1024^2                 1545, 1752
//      632   2025 on a 45 x 45 scan at 512^2          761, 806
//     1278   16,384 anywhere at 1024^2               5749, 5377
//   small sums do not pay for the launch: 4096 probes, 69 beams at 64^2 (2e9
//   operations) 31, 34; at 256^2 (6e10) 158, 152.
//   and full tiles of a part of S (n_tiles below those of the grid) count as the
//   others do: 8192 probes at one place, 1245 beams at 1024^2 (512) 2099, 2359;
//   16,384 within 5 of 100 A (1274) 7856, 6607.
inline bool bf16_records_route(int64_t n_entries, int64_t exact_entries, int64_t n_tiles, int64_t n_beams, int64_t ns) {
    const double products = (double)n_entries * 256, uses = products / ((double)ns * ns);
    const bool full = n_entries == exact_entries && n_tiles * 256 >= ns * ns;
    return uses >= (full ? 200 : 900) && products * 8 * n_beams >= 3e10;
}

}  // namespace prism
