// kernels.hpp -- host-side launchers of the gfx950 kernels (internal).
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace prism {

// Band-limited wave buffer layout used by the propagation passes:
//   W[item][j][y], j in [0, n/2) a band column (kx = j for j < n/4, j - n/2
//   otherwise), y in [0, n) the real-space row.  One "item" is a beam
//   (S-matrix) or a probe (multislice).  Columns are wave_col_stride(n) >= n
//   elements apart so that the column starts do not all fall on the same
//   power-of-two address stride at n = 2048 (row pass of 128 beams: 2.34 -> 2.10
//   ms with 256 bytes of padding; 64, 192 and 512 bytes or more: 2.12-2.19).  At
//   1024^2 the same padding gave 2% of the row pass (64 bytes: a quarter lost).
constexpr int wave_col_stride(int n) { return n >= 2048 ? n + 32 : n; }
struct PropTables {
    const float2* tw_half;   // W_{n/2}[m] = e^{-2 pi i m/(n/2)}, n/2 entries
    const float2* tw_full;   // W_n[m]     = e^{-2 pi i m/n},     n entries
    const float2* band_tw;   // e^{-2 pi i kx(j)/n}, n/2 entries
    const float2* prop;      // (1/n) e^{-i pi lambda dz kx(j)^2 / L^2}, n/2 entries
};

enum PassBMode { PASSB_MID = 0, PASSB_LAST_S = 1, PASSB_LAST_I = 2, PASSB_INIT = 3 };

// T[s][y][x] = exp(i sigma V[s][y][x]) for count = n_slices*n*n pixels.
hipError_t launch_transmission(const float* V, float2* T, int64_t count, float sigma, hipStream_t st);

// Row pass: for each item and real-space row y, inverse row transform of the
// band, multiply by T[y][x], forward row transform, keep the band.
hipError_t launch_pass_a(int n, float2* W, const float2* T, const PropTables& tb, int n_items, hipStream_t st);

// First row pass of plane-wave items, through the row spectrum of the first
// slice's transmission: R[c][y] = sum_x T0[y][x] e^{-2 pi i c x/n} (complex64
// [n][n], frequency-major), then W[item][j][y] = e^{2 pi i ky y/n}
// R[(kx(j) - kx) mod n][y] for the item's beam (kx, ky) -- the band of the
// row transform of the plane wave times T0.
hipError_t launch_row_spectrum(int n, const float2* T0, float2* R, const PropTables& tb, hipStream_t st);
hipError_t launch_first_from_spectrum(int n, float2* W, const float2* R, const PropTables& tb, const int2* beams,
                                      int n_items, hipStream_t st);

// Column pass (see PassBMode).  inten: band intensities [item][j][j'] for
// PASSB_LAST_I.  For PASSB_INIT the spectrum is the aperture: |ky| <= ky_max[j],
// coefficient amp e^{-2 pi i (kx x + ky y)/L} times aberr[j][j'] when `aux`
// (the aberration table, complex [n/2][n/2]) is not null.  `beside`: such launches
// at the same time (on other streams).
hipError_t launch_pass_b(int n, int mode, float2* W, const PropTables& tb, const float2* aux, float* inten,
                         const int* ky_max, const double2* probe_xy, double inv_L, float amp, int n_items,
                         hipStream_t st, int beside = 1);

// Final S-matrix pass: S[b][my][mx] = inverse row transform of half[b][j][my].
hipError_t launch_smatrix_final(int n, const float2* half, float2* S, const float2* tw_half, int n_items,
                                hipStream_t st);

// ---- projected potential --------------------------------------------------
// Atoms sorted by (slice, cell of a cells x cells grid over the wrapped
// positions, row-major); cell_start[(slice cells + cy) cells + cx] is a cell's
// first atom, with one more entry for the end.
struct PotAtom { double x, y; int32_t species, pad; };
struct PotSpecies { float amp_n[4]; float inv2w2[4]; float rc2; int n_gauss; float rc; int pad; };
hipError_t launch_potential(float* V, int n, int n_slices, double L, int cells, const PotAtom* atoms,
                            const int* cell_start, const PotSpecies* species, int max_gauss, float rc_max,
                            hipStream_t st);

// ---- probe synthesis ----------------------------------------------------------
// A K step of the contraction is 16 beams.
constexpr int KSTEP = 16;
inline int ksteps_of(int n_beams) { return (n_beams + KSTEP - 1) / KSTEP; }
// Bytes of the C operand, one record of up to 128 bytes per (probe, K step).
inline size_t c_operand_bytes(int64_t n_probes, int n_beams) { return (size_t)n_probes * ksteps_of(n_beams) * 128; }
// Coefficients amp * exp(-2 pi i (kx_b x_p + ky_b y_p) / L) (FP64 argument, range
// reduced), times aberr[b] when aberr is not null, as the C operand of `precision`.
hipError_t launch_coefficients(int precision, void* C, const double2* xy, const int2* beams, const float2* aberr,
                               int n_probes, int n_beams, double inv_L, float amp, hipStream_t st);

// Windowed contraction of one probe set: win[p][v][u] = sum_b C[p][b] S[b][pix]
// over the plan's work tiles (16 x 16 pixels from tile_origin, periodic).
// C is the precision's operand (launch_coefficients), S complex64
// [n_beams][ns][ns], or with `records` its BF16 records (PRISM_BF16, same sums).
struct ContractArgs {
    const void* C;
    const void* S;
    float2* win;
    const int* tile_start;
    const int* tile_probes;
    const int2* tile_origin;
    const int2* corner;
    int n_tiles, max_per_tile, n_beams, ns, m;
    int accumulate = 0;       // add to the windows (partial sums over beam chunks)
};
// Probes per workgroup of the contraction (the plan's work-tile cost unit).
int contract_probe_chunk();
// All jobs in as few launches as possible (one per 24 jobs).
hipError_t launch_contract_batch(int precision, const ContractArgs* jobs, int n_jobs, hipStream_t st, bool records = false);
size_t bf16_record_bytes(int n_beams, int ns);
hipError_t launch_bf16_records(const float2* S, void* records, int n_beams, int ns, hipStream_t st);

// The same windows by sums over kx, per distinct x of the probes ("scan
// column"), then over ky (PRISM_FP32 and PRISM_SPLIT_BF16X3).
struct TwoStageArgs {
    const float2* S;
    float2* T;                 // scratch of T_bytes, at least one column's
    size_t T_bytes;
    float2* win;
    void *cx, *cy;             // C operands, two_stage_cx_bytes and two_stage_cy_bytes
    const double2 *col_xy, *xy;   // (x, 0) of each column; probe positions
    const int2* beams;
    const float2* aberr;
    const int4* steps;         // per K step of a column (beams of one ky): first beam, beams, ky row, last of its ky
    const int4* rows;          // per ky: first beam, beams, first K step, ky
    const int *col_corner, *col_start, *entry_corner, *entry_probe;   // see struct TwoStage
    int n_cols, col_steps, n_probes, n_rows, ns, m;
    int max_row_beams;         // most beams of one ky
    int tile_width;            // of the first sum's 128-pixel tiles
    int max_cols, max_probes;  // most columns over tile_width pixels; most probes of a column over the
                               // rows of 128 window pixels
    double inv_L;
    float amp;
};
size_t two_stage_cx_bytes(int n_cols, int col_steps);
size_t two_stage_cy_bytes(int64_t n_probes, int n_rows);
size_t two_stage_column_bytes(int n_rows, int ns, int m);
hipError_t launch_two_stage_operands(const TwoStageArgs& t, hipStream_t st);
// Scan columns per pair of launches (whose T fits), and the two sums for
// columns q0 .. q0 + n - 1.
int two_stage_columns(const TwoStageArgs& t);
// Workgroups of both sums' launches over the first columns, or -1 when a launch
// does not hold them (every column gets as many as the one with most probes).
int64_t two_stage_blocks(const TwoStageArgs& t);
hipError_t launch_sum_kx(int precision, const TwoStageArgs& t, int q0, int n, hipStream_t st);
hipError_t launch_sum_ky(const TwoStageArgs& t, int q0, int n, hipStream_t st);

// out[p][bin] = sum over the bin's pixels of |FFT_m(win[p])|^2 / m^4.  For
// m > 128 the window is transformed in place and `inten` ([p][m*m] floats)
// holds the intensities; for m <= 128 both stay untouched.
struct WindowArgs {
    float2* win;
    float* inten;
    float* out;                // binned output, or null
    float* diff;               // [p][m][m] intensities (4D output), or null
    const int* perm;
    const int* bin_start;
    const float2* tw_m;
    int n_probes, n_bins;
    float scale;               // binned output = scale * sum (+ previous value when accumulating)
    int accumulate;
};
// All jobs of one window side m (one launch per 24 jobs for m <= 128).
hipError_t launch_window_batch(int m, const WindowArgs* jobs, int n_jobs, hipStream_t st);

// out[p][bin] = sum over bin pixels of inten[p][pix] (deterministic order).
hipError_t launch_bin_reduce(const float* inten, int64_t pix_per_item, float* out, const int* perm,
                             const int* bin_start, int n_items, int n_bins, hipStream_t st, float scale = 1.f,
                             int accumulate = 0);

}  // namespace prism
