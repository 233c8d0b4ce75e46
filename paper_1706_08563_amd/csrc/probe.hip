// probe.hip -- PRISM probe synthesis: coefficients, windowed beam contraction,
// window FFT with |Psi|^2, and deterministic annular-detector sums.
//
// "PRISM Probe Simulations": each probe is a sum over plane waves of the
// cropped S-matrix layers times per-beam phase coefficients; the modulus
// squared of the FFT of that exit wave is binned into detectors (Fig. 1i-k).
#include "fft.hpp"
#include "kernels.hpp"
#include "launch_limits.hpp"

#include <algorithm>
#include <type_traits>

namespace prism {

constexpr int WG = 256;

// ------------------------------------------------------------ coefficients --
// C[p][b] = amp e^{-2 pi i (kx x + ky y)/L}; the phase argument is formed in
// FP64 and reduced to [-1/2, 1/2] turns before the FP32 sincos.
__device__ __forceinline__ float2 coefficient(double2 r, int2 k, const float2* __restrict__ aberr, int b,
                                              double inv_L, float amp) {
    double a = ((double)k.x * r.x + (double)k.y * r.y) * inv_L;
    float fr = (float)(a - rint(a));
    float s, c;
    sincosf(-6.283185307179586f * fr, &s, &c);
    float2 v = make_float2(amp * c, amp * s);
    if (aberr) v = cmul(v, aberr[b]);
    return v;
}

// --------------------------------------------------- windowed contraction --
// The contraction runs over work tiles of 16 x 16 S-grid pixels.  A probe's
// M x M window starts at its corner; the plan gives every probe a tiling
// phase (an offset of the 16-pixel tile grid, at most its corner's position
// modulo 16) and lists the probe under each tile of that phase its window
// overlaps.  When the phase equals the corner's offset (as for probes on a
// scan lattice of a few pixels' pitch) the window is exactly (M/16)^2 tiles and
// no product falls outside it.  A workgroup takes one work tile and a chunk
// of PC of its probes and forms, for every tile pixel,
//     acc[p] = sum_b C[p][b] S[b][pixel]
// then stores each (probe, pixel) that lies inside the probe's window.  The
// tiles of one phase partition the S grid, so each window element is
// produced by exactly one (tile, probe) pair: no atomics.
constexpr int TILE = 16;

// Work of one (request's) probe synthesis inside a batched contraction launch.
struct ContractJob {
    const void* C;            // coefficients (k_coefficients)
    const void* S;            // S-matrix: complex64 [n_beams][ns][ns], or its BF16 records
    float2* win;              // [n_probes][m][m]
    const int* tile_start;    // [n_tiles + 1]
    const int* tile_probes;
    const int2* tile_origin;  // [n_tiles] first pixel (x, y) of each work tile
    const int2* corner;       // window corner per probe
    int n_beams, ns, m;
    int ksteps;               // K steps of 16 beams
    int accumulate;           // 1: add to the windows' contents (beam chunks of one sum)
    int chunks;               // workgroups per tile
    int n_tiles;
    int block0;               // first logical workgroup of this job
};
constexpr int MAX_JOBS = 24;
struct ContractBatch {
    int n_jobs;
    int n_blocks;             // logical workgroups over all jobs
    int per_xcd;              // logical workgroups per XCD slot
    ContractJob job[MAX_JOBS];
};

// Logical workgroup of this hardware workgroup.  Hardware workgroups are
// dealt round-robin to the 8 XCDs; consecutive logical workgroups are placed
// on the same XCD, so the probe chunks and phases of neighbouring tiles (the
// plan orders work tiles by position, then phase) share that XCD's L2.
// The selected job is copied out by value: taking the address of the
// by-value kernel argument would force a private-memory copy of the table.
__device__ __forceinline__ bool locate(const ContractBatch& b, ContractJob& job, int& tile, int& chunk) {
    const int hw = blockIdx.x;
    const int l = (hw & 7) * b.per_xcd + (hw >> 3);
    if (l >= b.n_blocks) return false;
    int j = 0;
#pragma unroll
    for (int k = 1; k < MAX_JOBS; ++k)
        if (k < b.n_jobs && b.job[k].block0 <= l) j = k;
    job = b.job[j];
    const int local = l - job.block0;
    tile = local / job.chunks;
    chunk = local % job.chunks;
    return true;
}

// The complex product is carried by real BF16 MFMA (v_mfma_f32_32x32x16_bf16,
// FP32 accumulators) over K = 8 beams x (re, im), interleaved: with operand
// words (re | im << 16),
//   Re = (Cr, -Ci) . (Sr, Si)        Im = (Ci, Cr) . (Sr, Si)
// so both need one S operand, and the two C operands are a sign flip and a
// half-word rotation of the stored word.
//
// An FP32 operand is a sum of NP BF16 parts, each the rounding of what the
// parts before it leave (the differences are exact):
//   NP = 3 (FP32)   all 24 bits; products hh, hm, mh, mm, hl, lh.  What is
//                   left out (ml, lm, ll) is at most 2^-24 of the product in
//                   all, as much as the rounding of an FP32 product.
//   NP = 2 (split)  16 bits; hh, hl, lh (lo lo, ~2^-16 relative, left out).
//   NP = 1 (BF16)   hh.
//
// A workgroup is one work tile (or half of one) x PC = 64 probes: a wave
// owns CB 32-pixel column blocks, 2 CB tile rows, and all probes (two 32-row
// blocks).  A lane's S operand of a step of 8 beams is 4 beams of one pixel,
// which it loads itself (no other wave needs them: nothing goes through LDS)
// two steps ahead and converts in registers.  C of 16 beams x 64 probes is
// shared through a double-buffered LDS tile [part][4-beam group][probe], one
// barrier per 16 beams.
//
// Bound: MFMA power.  16,384 probes x 1245 beams x 128^2 windows in split
// BF16 take 7.0 ms: 1.15 PFLOP/s of MFMA work at the 1.5 GHz the clock drops
// to, the rate of a large library BF16 product on the same card (1.18).
// Before: S converted to BF16 records by a pass of its own (1.06 ms, and as
// much memory again as S) and both operands staged through LDS, 6.8 + 1.06
// ms; with few probes per pixel the pass was as long as the contraction (441
// probes of 256^2 windows: 1.16 + 1.07 -> 1.02 ms).  Plain BF16 reads such records
// where sums are large (k_bf16_records).  FP32 products on the
// VALU: 2025 probes x 1245 beams x 128^2, 7.1 -> 2.0 ms with six BF16 products.
namespace mfmac {
constexpr int NT = 256;               // threads per workgroup
constexpr int PC = SUM_ROWS;          // probes per workgroup
constexpr int RB = PC / 32;           // 32-probe row blocks
constexpr int SUB = SUM_PLANES;       // beams per MFMA step, half a K step
// A wave owns CB = 1 or 2 32-pixel column blocks (pairs of tile rows); with one,
// two workgroups share a tile.  FP32 takes one, so that the registers of the
// other hold the sum of the last FLUSH K steps apart from the running total: an
// FP32 sum of 1245 beams, 6 products each, is otherwise rounded 936 times at the
// size of the total (2025 probes of 1245 beams: error against 64 bits 1.4e-7 on
// the VALU, 1.7e-7 without the split total, 9e-8 with it).  The other precisions
// take two from MIN_BLOCKS workgroups on and one below, where two leave CUs with
// little to do (same sums, same bits).  Split BF16, one and two: 256 probes of 69
// beams at 256^2, the whole call, 36 and 44 us; 1600 of 305 beams at 512^2 109 and
// 119; 3600 of 1245 beams at 1024^2 2.45 and 2.42 ms; 16,384 10.0 and 9.5 ms.
constexpr int MIN_BLOCKS = 1024;
template <int NP> constexpr int FLUSH = NP == 3 ? 2 : 1 << 30;
}

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

// Two floats to packed bf16 (round to nearest even, v_cvt_pk_bf16_f32).
__device__ __forceinline__ unsigned int pack_bf16(float a, float b) {
    bf16x2 h = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(unsigned int, h);
}
__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// The NP parts of one complex value, as words (re | im << 16).
template <int NP>
__device__ __forceinline__ void split_parts(float re, float im, unsigned int (&w)[NP]) {
#pragma unroll
    for (int part = 0; part < NP; ++part) {
        w[part] = pack_bf16(re, im);
        re -= __uint_as_float(w[part] << 16);
        im -= __uint_as_float(w[part] & 0xffff0000u);
    }
}

// C operands, thread = (row, group of 4 beams): split records
// [row][K step][part][4-beam group] for NP = 1, 2, and the FP32 values
// [row][K step][16 beams] (the same bytes as NP = 2) for NP = 3, which the
// contraction splits as it stages them.  Beams past the last are zero.  A row
// is a probe, or a scan column of the two-stage sum.
template <int NP> constexpr int REC = NP == 3 ? 8 : NP * 4;   // 16-byte words per record
template <int NP>
__device__ __forceinline__ void store_operand(u32x4* rec, int g, const float2 (&v)[4]) {
    if constexpr (NP == 3) {
        float4* dst = reinterpret_cast<float4*>(rec) + 2 * g;
        dst[0] = make_float4(v[0].x, v[0].y, v[1].x, v[1].y);
        dst[1] = make_float4(v[2].x, v[2].y, v[3].x, v[3].y);
    } else {
        u32x4 ch[NP];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            unsigned int w[NP];
            split_parts<NP>(v[j].x, v[j].y, w);
#pragma unroll
            for (int part = 0; part < NP; ++part) ch[part][j] = w[part];
        }
#pragma unroll
        for (int part = 0; part < NP; ++part) rec[part * 4 + g] = ch[part];
    }
}

template <int NP>
__global__ __launch_bounds__(WG) void k_coefficients(u32x4* __restrict__ C, const double2* __restrict__ xy,
                                                     const int2* __restrict__ beams,
                                                     const float2* __restrict__ aberr, int n_probes, int n_beams,
                                                     int K, double inv_L, float amp) {
    const int64_t total = (int64_t)n_probes * K * 4;
    for (int64_t i = (int64_t)blockIdx.x * WG + threadIdx.x; i < total; i += (int64_t)gridDim.x * WG) {
        const int p = (int)(i / (4 * K)), r = (int)(i % (4 * K)), k = r >> 2, g = r & 3;
        const double2 xyp = xy[p];
        float2 v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int b = k * KSTEP + g * 4 + j;
            v[j] = b < n_beams ? coefficient(xyp, beams[b], aberr, b, inv_L, amp) : make_float2(0.f, 0.f);
        }
        store_operand<NP>(C + (i >> 2) * REC<NP>, g, v);
    }
}

hipError_t launch_coefficients(int precision, void* C, const double2* xy, const int2* beams, const float2* aberr,
                               int n_probes, int n_beams, double inv_L, float amp, hipStream_t st) {
    const int K = ksteps_of(n_beams);
    const int64_t total = (int64_t)n_probes * K * 4;
    int64_t blocks = (total + WG - 1) / WG;
    if (blocks > 65536) blocks = 65536;
    if (blocks < 1) blocks = 1;
    u32x4* Cw = static_cast<u32x4*>(C);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(WG), 0, st, Cw, xy, beams, aberr, n_probes, n_beams, K,
                           inv_L, amp);
    };
    if (precision == 0)
        launch(k_coefficients<3>);
    else if (precision == 1)
        launch(k_coefficients<2>);
    else
        launch(k_coefficients<1>);
    return hipGetLastError();
}

// S as BF16 records, 32 bytes per (step of 8 beams, pixel): the words (re | im <<
// 16) of its beams, zero past the last.  A thread makes one record, a wave 2 KB.
// For large sums in plain BF16 (bf16_records_route): a lane's operand of a step is
// then one load of 16 bytes in runs of 512, where S takes four of 8 in runs of
// 128, most of which lie across two lines.  Bound: HBM traffic, S read and half as
// much written (1245 beams at 1024^2 0.66 ms, 5.9 TB/s).  16,384 probes of 128^2:
// contraction 4.9 -> 3.1 ms, the call 5.8 -> 4.4.
__global__ __launch_bounds__(WG) void k_bf16_records(const float2* __restrict__ S, u32x4* __restrict__ rec, int n_beams,
                                                     int plane) {
    const int pix = blockIdx.x * WG + threadIdx.x, step = blockIdx.y;
    if (pix >= plane) return;
    u32x4 w[2];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int b = step * 8 + j;
        const float2 v = b < n_beams ? S[(size_t)b * plane + pix] : make_float2(0.f, 0.f);
        w[j / 4][j % 4] = pack_bf16(v.x, v.y);
    }
    u32x4* out = rec + ((size_t)step * plane + pix) * 2;
    out[0] = w[0];
    out[1] = w[1];
}

size_t bf16_record_bytes(int n_beams, int ns) { return (size_t)ksteps_of(n_beams) * KSTEP * ns * ns * 4; }
hipError_t launch_bf16_records(const float2* S, void* records, int n_beams, int ns, hipStream_t st) {
    const int plane = ns * ns;
    hipLaunchKernelGGL(k_bf16_records, dim3((unsigned)((plane + WG - 1) / WG), 2u * ksteps_of(n_beams)), dim3(WG), 0, st, S,
                       static_cast<u32x4*>(records), n_beams, plane);
    return hipGetLastError();
}

// LDS of a contraction workgroup, C operand in NA parts.
template <int NA>
struct ContractLds {
    static constexpr int NCH = NA * 4;            // 16-byte chunks of a K step's operand row
    // row stride of a chunk: odd (or = 2 mod 8 when 4 lanes write one row) so
    // that 8 lanes of a staging store hit distinct bank groups
    static constexpr int LP = NA == 3 ? mfmac::PC + 2 : mfmac::PC + 1;
    u32x4 C[2][NCH * LP];
    int idx[mfmac::PC];                           // C operand of each row, or -1
    int2 at[mfmac::PC];                           // window corner of each row
};
// Row (MFMA row: probe or scan column) of D register r of row block rb.
__device__ __forceinline__ int sum_row(int rb, int r, int half) { return 32 * rb + (r & 3) + 8 * (r >> 2) + 4 * half; }

// Registers and steps of the pipelined product of C (NA parts, through LDS)
// and S (NB parts, CB 32-pixel column blocks of the wave).  RECS: S comes as the
// BF16 records of k_bf16_records instead of complex64 planes.
template <int NA, int NB, int CB, bool RECS = false>
struct BeamPipe {
    static_assert(!RECS || NB == 1, "records hold one part");
    static constexpr int NCH = NA * 4, LP = ContractLds<NA>::LP, NT = mfmac::NT;
    static constexpr int CW = NA == 3 ? 2 : NA, NCP = NA == 3 ? 1 : NA;
    static constexpr int NL = RECS ? 1 : 4;       // loads of a lane's 4 beams
    using Raw = std::conditional_t<RECS, u32x4, float2>;
    int voff[CB][NL];
    Raw raw[2][CB][NL];                           // S of the two halves of a K step, in flight
    u32x4 B[2][NB][CB];                           // the same converted
    u32x4 creg[CW];
    const u32x4* cptr[NCP];

    // S operand of this lane: pixel pix[cb] of column block cb, beams 4 half
    // .. 4 half + 3 of a step; byte offsets from the start of the step.
    // C staging.  NA <= 2: chunk (tid + j NT) of a K step's PC records;
    // NA = 3: the 4 beams (tid % 4) of row tid / 4, split when stored.
    // Rows without an operand (idx < 0) read operand 0; nothing of them is stored.
    __device__ __forceinline__ void init(const ContractLds<NA>& lds, const int (&pix)[CB], int plane_bytes,
                                         const u32x4* C, int stride) {
        const int tid = threadIdx.x, half = (tid & 63) >> 5;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int j = 0; j < NL; ++j)
                voff[cb][j] = RECS ? (2 * pix[cb] + half) * (int)sizeof(u32x4)
                                   : pix[cb] * (int)sizeof(float2) + (4 * half + j) * plane_bytes;
#pragma unroll
        for (int j = 0; j < NCP; ++j) {
            const int q = max(lds.idx[NA == 3 ? tid / 4 : (tid + j * NT) / NCH], 0);
            const int off = NA == 3 ? (tid % 4) * 2 : (tid + j * NT) % NCH;
            cptr[j] = C + (size_t)q * stride * REC<NA> + off;
        }
    }
    // Buffer loads from a scalar resource that ends with the last beam (left
    // bytes from the start of the step), so that beams past it read as zero
    // and the loop holds no branch around a load (each would end in a wait
    // for all loads in flight).
    __device__ __forceinline__ void load_s(int h, const void* S, int64_t left) {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<void*>(S), (short)0, (int)max((int64_t)0, min(left, MAX_BUFFER_BYTES)), 0x00020000);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int j = 0; j < NL; ++j) {
                if constexpr (RECS)
                    raw[h][cb][j] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, voff[cb][j], 0, 0));
                else
                    raw[h][cb][j] = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rs, voff[cb][j], 0, 0));
            }
    }
    __device__ __forceinline__ void convert_s(int h) {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            if constexpr (RECS) {
                B[h][0][cb] = raw[h][cb][0];
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    unsigned int w[NB];
                    split_parts<NB>(raw[h][cb][j].x, raw[h][cb][j].y, w);
#pragma unroll
                    for (int part = 0; part < NB; ++part) B[h][part][cb][j] = w[part];
                }
            }
        }
    }
    // Ends the conversion of half h here (not sunk to where its results are
    // used): the loads that follow reuse its registers and are not moved down.
    __device__ __forceinline__ void pin(int h) {
#pragma unroll
        for (int part = 0; part < NB; ++part)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) asm volatile("" : "+v"(B[h][part][cb]));
        __builtin_amdgcn_sched_barrier(0);
    }
    __device__ __forceinline__ void load_c(int step) {
        const size_t at = (size_t)step * REC<NA>;
#pragma unroll
        for (int j = 0; j < CW; ++j) creg[j] = NA == 3 ? cptr[0][at + j] : cptr[NA == 3 ? 0 : j][at];
    }
    __device__ __forceinline__ void stage_c(u32x4* dst) const {
        const int tid = threadIdx.x;
        if constexpr (NA == 3) {
            u32x4 ch[3];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                unsigned int w[3];
                split_parts<3>(__uint_as_float(creg[j / 2][(j % 2) * 2]), __uint_as_float(creg[j / 2][(j % 2) * 2 + 1]), w);
#pragma unroll
                for (int part = 0; part < 3; ++part) ch[part][j] = w[part];
            }
#pragma unroll
            for (int part = 0; part < 3; ++part) dst[(part * 4 + tid % 4) * LP + tid / 4] = ch[part];
        } else {
#pragma unroll
            for (int j = 0; j < CW; ++j) dst[((tid + j * NT) % NCH) * LP + (tid + j * NT) / NCH] = creg[j];
        }
    }
    // Products of half h of the K step staged in Ck with row block rb.
    __device__ __forceinline__ void products(const u32x4* Ck, int h, int rb, f32x16 (&accr)[CB], f32x16 (&acci)[CB]) const {
        const int lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
        u32x4 A[NA];
#pragma unroll
        for (int part = 0; part < NA; ++part) A[part] = Ck[(part * 4 + 2 * h + half) * LP + 32 * rb + col];
        auto product = [&](f32x16 (&acc)[CB], int pa, int pb) {
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
                acc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(A[pa]), as_bf16x8(B[h][pb][cb]), acc[cb], 0, 0, 0);
        };
        auto all = [&](f32x16 (&acc)[CB]) {
            if constexpr (NA == 3) product(acc, 2, 0);
            if constexpr (NB == 3) {
                product(acc, 0, 2);
                product(acc, 1, 1);
            }
            if constexpr (NA >= 2) product(acc, 1, 0);
            if constexpr (NB >= 2) product(acc, 0, 1);
            product(acc, 0, 0);
        };
#pragma unroll
        for (int part = 0; part < NA; ++part) A[part] ^= 0x80000000u;             // (Cr, -Ci)
        all(accr);
#pragma unroll
        for (int part = 0; part < NA; ++part) {                                   // (Ci, Cr)
            A[part] ^= 0x80000000u;
            A[part] = (A[part] >> 16) | (A[part] << 16);
        }
        all(acci);
    }
};
template <int RB, int CB>
__device__ __forceinline__ void clear(f32x16 (&a)[RB][CB]) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int r = 0; r < 16; ++r) a[rb][cb][r] = 0.f;
}
template <int CB>
struct Sums {
    f32x16 r[mfmac::RB][CB], i[mfmac::RB][CB];
};

// sum[row][pixel] = sum over the n_beams planes of S (plane elements apart)
// of C[lds.idx[row]][beam] S[beam][pix]: one lane's pixels are pix[cb]; C rows
// are `stride` records apart; `two`: the second row block holds rows; every
// FLUSH K steps are summed by themselves.  Called by all threads of the
// workgroup, lds.idx written and synchronised.  RECS: S as BF16 records.
template <int NP, int CB, int FLUSH, bool RECS = false>
__device__ __forceinline__ void sum_beams(ContractLds<NP>& lds, const void* __restrict__ S, size_t plane, int n_beams,
                                          const int (&pix)[CB], const u32x4* __restrict__ C, int stride, bool two,
                                          Sums<CB>& sum) {
    using namespace mfmac;
    const int K = (n_beams + KSTEP - 1) / KSTEP, plane_bytes = (int)(plane * sizeof(float2));
    constexpr bool PARTS = FLUSH < 1 << 30;
    f32x16 accr[RB][CB], acci[RB][CB];
    clear(accr);
    clear(acci);
    if constexpr (PARTS) {
        clear(sum.r);
        clear(sum.i);
    }
    BeamPipe<NP, NP, CB, RECS> pipe;
    pipe.init(lds, pix, plane_bytes, C, stride);
    auto load_s = [&](int k, int h) {
        if constexpr (RECS) {
            const int step = min(2 * k + h, 2 * K - 1);
            pipe.load_s(h, static_cast<const u32x4*>(S) + (size_t)step * plane * 2, (int64_t)plane * 32);
        } else {
            const int b0 = min(k * KSTEP + h * SUB, n_beams);
            pipe.load_s(h, static_cast<const float2*>(S) + (size_t)b0 * plane, (int64_t)(n_beams - b0) * plane_bytes);
        }
    };
    pipe.load_c(0);
    load_s(0, 0);
    load_s(0, 1);
    pipe.stage_c(lds.C[0]);
    __syncthreads();
    // step s + 1 is converted while the products of step s run
    pipe.convert_s(0);
    load_s(1, 0);
    for (int k0 = 0; k0 < K; k0 += FLUSH) {
        const int k1 = min(k0 + FLUSH, K);
        for (int k = k0; k < k1; ++k) {
            pipe.load_c(min(k + 1, K - 1));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                pipe.convert_s(1 - h);
                pipe.products(lds.C[k & 1], h, 0, accr[0], acci[0]);
                pipe.pin(1 - h);
                load_s(h == 0 ? k + 1 : k + 2, 1 - h);
                __builtin_amdgcn_sched_barrier(0);
                if (two) pipe.products(lds.C[k & 1], h, 1, accr[1], acci[1]);
            }
            pipe.stage_c(lds.C[(k + 1) & 1]);
            __syncthreads();
        }
        if constexpr (PARTS) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) {
                    sum.r[rb][cb] += accr[rb][cb];
                    sum.i[rb][cb] += acci[rb][cb];
                }
            clear(accr);
            clear(acci);
        }
    }
    if constexpr (!PARTS) {
#pragma unroll
        for (int a = 0; a < RB; ++a)
#pragma unroll
            for (int b = 0; b < CB; ++b) {
                sum.r[a][b] = accr[a][b];
                sum.i[a][b] = acci[a][b];
            }
    }
}

template <int NP, int CB, bool RECS = false>
__global__ __launch_bounds__(mfmac::NT) __attribute__((amdgpu_waves_per_eu(2))) void k_contract(ContractBatch batch) {
    using namespace mfmac;
    constexpr int SPLITS = 2 / CB;                    // workgroups per (tile, probe chunk)
    __shared__ ContractLds<NP> lds;
    int tile, chunk;
    ContractJob job;
    if (!locate(batch, job, tile, chunk)) return;
    const int row0 = 8 * CB * (chunk % SPLITS);   // first tile row of this workgroup
    chunk /= SPLITS;
    float2* __restrict__ win = job.win;
    const int ns = job.ns, m = job.m;
    const int t0 = job.tile_start[tile], t1 = job.tile_start[tile + 1];
    const int pc0 = t0 + chunk * PC;
    if (pc0 >= t1) return;
    const int np = min(PC, t1 - pc0);
    const int2 org = job.tile_origin[tile];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int col = lane & 31, half = lane >> 5;
    if (tid < PC) {
        const int q = tid < np ? job.tile_probes[pc0 + tid] : -1;
        lds.idx[tid] = q;
        lds.at[tid] = q >= 0 ? job.corner[q] : make_int2(0, 0);
    }
    __syncthreads();
    int px = (org.x + (col & 15)) & (ns - 1), py[CB], pix[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
        py[cb] = (org.y + row0 + 2 * (CB * wave + cb) + (col >> 4)) & (ns - 1);
        pix[cb] = py[cb] * ns + px;
    }
    Sums<CB> sum;
    sum_beams<NP, CB, FLUSH<NP>, RECS>(lds, job.S, (size_t)ns * ns, job.n_beams, pix, static_cast<const u32x4*>(job.C),
                                 job.ksteps, np > 32, sum);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = sum_row(rb, r, half);
            const int q = lds.idx[row];
            if (q < 0) continue;
            const int2 c0 = lds.at[row];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                const int v = (py[cb] - c0.y) & (ns - 1);
                const int u = (px - c0.x) & (ns - 1);
                if (v < m && u < m) {
                    float2* w = win + (size_t)q * m * m + (size_t)v * m + u;
                    float2 res = make_float2(sum.r[rb][cb][r], sum.i[rb][cb][r]);
                    if (job.accumulate) res = cadd(*w, res);
                    *w = res;
                }
            }
        }
}

int contract_probe_chunk() { return mfmac::PC; }

hipError_t launch_contract_batch(int precision, const ContractArgs* jobs, int n_jobs, hipStream_t st, bool records) {
    for (int j0 = 0; j0 < n_jobs; j0 += MAX_JOBS) {
        ContractBatch b{};
        b.n_jobs = n_jobs - j0 < MAX_JOBS ? n_jobs - j0 : MAX_JOBS;
        auto chunks_of = [](const ContractArgs& a) { return std::max(1, (a.max_per_tile + mfmac::PC - 1) / mfmac::PC); };
        int64_t whole = 0;                                // workgroups with two column blocks
        for (int k = 0; k < b.n_jobs; ++k) whole += (int64_t)chunks_of(jobs[j0 + k]) * jobs[j0 + k].n_tiles;
        const bool two = precision != 0 && whole >= mfmac::MIN_BLOCKS;
        int blocks = 0;
        for (int k = 0; k < b.n_jobs; ++k) {
            const ContractArgs& a = jobs[j0 + k];
            ContractJob& job = b.job[k];
            job.C = a.C;
            job.S = a.S;
            job.win = a.win;
            job.tile_start = a.tile_start;
            job.tile_probes = a.tile_probes;
            job.tile_origin = a.tile_origin;
            job.corner = a.corner;
            job.n_beams = a.n_beams;
            job.ns = a.ns;
            job.m = a.m;
            job.ksteps = ksteps_of(a.n_beams);
            job.accumulate = a.accumulate;
            job.chunks = chunks_of(a) * (two ? 1 : 2);
            job.n_tiles = a.n_tiles;
            job.block0 = blocks;
            blocks += job.chunks * job.n_tiles;
        }
        b.n_blocks = blocks;
        b.per_xcd = (blocks + 7) / 8;
        if (blocks == 0) continue;
        dim3 grid((unsigned)(8 * b.per_xcd));
        auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(mfmac::NT), 0, st, b); };
        if (precision == 0)
            launch(k_contract<3, 1>);
        else if (precision == 1)
            two ? launch(k_contract<2, 2>) : launch(k_contract<2, 1>);
        else if (records)
            two ? launch(k_contract<1, 2, true>) : launch(k_contract<1, 1, true>);
        else
            two ? launch(k_contract<1, 2>) : launch(k_contract<1, 1>);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// --------------------------------------------------------- two-stage sum --
// A coefficient is a product of one phase per axis, and the probes of a scan
// share few x positions, so the beam sum splits into
//   T[x][ky][pixel] = sum_kx c_b(x) S_b[pixel]      (aberrations, amplitude)
//   win[probe][pixel] = sum_ky e^{-2 pi i ky y / L} T[x][ky][pixel]
// with (for 16,384 probes of 1245 beams) a sixteenth of the products.  T is
// kept for the columns of the windows at x only: [ky][S-grid row][x][window
// column] (x next to the window column, so that a tile's writes for all its x
// spread over the memory channels).  Scan columns are sorted by window corner, and the probes of each
// by corner too, so those whose windows cover a tile are one cyclic run.
//
// Bound: HBM traffic (S read, T written and read, windows written) and the
// latency of its short sums.  16,384 probes of 1245 beams, 128^2 windows at
// 1024^2, split BF16: 7.0 ms in one stage, 1.2 + 1.1 ms in two (10.4 GB, 4.5
// TB/s), with the products of the second stage in FP32 accuracy: the error
// against 64 bits falls from 7e-7 to 2.4e-7.  With T by [x][ky][row][column]
// and 16-pixel tiles the first stage took 1.9 ms.
struct TwoStage {
    const float2* S;
    float2* T;                // [n_rows][ns][columns of this launch][m]
    float2* win;              // [n_probes][m][m]
    const u32x4* cx;          // C operand of the launch's columns over their K steps
    const u32x4* cy;          // C operand of the probes over ky
    const int4* rows;         // per ky: first beam, beams, first K step, ky
    const int4* steps;        // per K step: first beam, beams, ky row, last of its ky
    const int* col_corner;    // window corner x of the launch's columns, ascending
    const int* col_start;     // first entry of each of the launch's columns, and the end
    const int* entry_corner;  // window corner y, ascending within a column
    const int* entry_probe;
    int n_cols, n_rows, col_steps, ns, m;
    int tile_width;           // of the first stage's 128-pixel tiles
    int row_groups;           // workgroups that share a tile's ky rows
    int chunks;               // workgroups per 64 scan columns / probes
    int n_blocks, per_xcd;
};

// Values of the sorted c[0 .. n) below x: each round narrows to a 64th.
__device__ __forceinline__ int lower_bound(const int* __restrict__ c, int n, int x) {
    const int lane = threadIdx.x & 63;
    int lo = 0, hi = n;
    while (lo < hi) {
        const int step = (hi - lo + 63) / 64, at = lo + lane * step;
        const int below = __popcll(__ballot(at < hi && c[at] < x));
        hi = min(hi, lo + below * step);
        lo = below ? lo + (below - 1) * step + 1 : hi;
    }
    return lo;
}

// The sorted corners c[0 .. n) whose windows of side m (cyclic on ns) cover
// any of `span` pixels from `from`: the cyclic run first, count.  Up to 256 are
// tested one by one, both counts in one pass over them; the search is for long
// columns (16,384 probes at one x, 64^2 windows at 256^2, the whole call: 1.21 ms
// one by one, 0.35 by search; 16,384 of 128^2 at 1024^2 5.0 and 1.8 ms).
__device__ __forceinline__ void cover_run(const int* __restrict__ c, int n, int from, int span, int m, int ns, int& first,
                                          int& count) {
    const int lane = threadIdx.x & 63, a = (from - (m - 1)) & (ns - 1), len = min(m + span - 1, ns);
    int below = 0, in = 0;
    if (n <= 256) {
        for (int base = 0; base < n; base += 64) {
            const bool have = base + lane < n;
            const int v = have ? c[base + lane] : 0;
            below += __popcll(__ballot(have && v < a));
            in += __popcll(__ballot(have && ((v - a) & (ns - 1)) < len));
        }
    } else {
        below = lower_bound(c, n, a);
        in = a + len <= ns ? lower_bound(c, n, a + len) - below : n - below + lower_bound(c, n, a + len - ns);
    }
    first = below == n ? 0 : below;
    count = in;
}

// T of 128 pixels (tile_width x 128 / tile_width rows), 64 scan columns and a
// run of ky.  The K steps of the run are one pipeline: the sum of a ky is
// stored while the loads of the next are in flight.  The C operand keeps all
// its parts also when S has two (NB): a column's operand is the same for every
// ky, and its rounding would add up over them (1.5 times the error of the
// one-stage sum).
constexpr int MAX_STEPS = 256;   // K steps of one workgroup
template <int NB>
__global__ __launch_bounds__(mfmac::NT) __attribute__((amdgpu_waves_per_eu(2))) void k_sum_kx(TwoStage a) {
    using namespace mfmac;
    __shared__ ContractLds<3> lds;
    __shared__ int4 step[MAX_STEPS];              // first beam, beams, ky row, last of its ky
    int l = (blockIdx.x & 7) * a.per_xcd + (blockIdx.x >> 3);
    if (l >= a.n_blocks) return;
    const int rg = l % a.row_groups;
    l /= a.row_groups;
    const int chunk = l % a.chunks;
    l /= a.chunks;
    const int ns = a.ns, m = a.m, tw = a.tile_width, nt = ns / tw;
    const int ox = l % nt * tw, oy = l / nt * (128 / tw);
    int first, count;
    cover_run(a.col_corner, a.n_cols, ox, tw, m, ns, first, count);
    const int np = min(PC, count - chunk * PC);
    if (np <= 0) return;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, col = lane & 31, half = lane >> 5;
    const int r0 = rg * a.n_rows / a.row_groups, r1 = (rg + 1) * a.n_rows / a.row_groups;
    const int t0 = a.rows[r0].z, n_steps = (r1 < a.n_rows ? a.rows[r1].z : a.col_steps) - t0;
    for (int t = tid; t < n_steps; t += NT) step[t] = a.steps[t0 + t];
    if (tid < PC) {
        const int q = tid < np ? (first + chunk * PC + tid) % a.n_cols : -1;
        lds.idx[tid] = q;
        lds.at[tid] = make_int2(q >= 0 ? a.col_corner[q] : 0, 0);
    }
    __syncthreads();
    const int at = wave * 32 + col, px = ox + at % tw, py = oy + at / tw;
    const int pix[1] = {py * ns + px};
    const size_t plane = (size_t)ns * ns;
    const int plane_bytes = (int)(plane * sizeof(float2));
    BeamPipe<3, NB, 1> pipe;
    pipe.init(lds, pix, plane_bytes, a.cx + (size_t)t0 * REC<3>, a.col_steps);
    auto load_s = [&](int t, int h) {
        const int4 s = step[min(t, n_steps - 1)];
        const int b0 = __builtin_amdgcn_readfirstlane(s.x) + h * SUB, nb = __builtin_amdgcn_readfirstlane(s.y) - h * SUB;
        pipe.load_s(h, a.S + (size_t)b0 * plane, (int64_t)nb * plane_bytes);
    };
    f32x16 accr[RB][1], acci[RB][1];
    clear(accr);
    clear(acci);
    pipe.load_c(0);
    load_s(0, 0);
    load_s(0, 1);
    pipe.stage_c(lds.C[0]);
    __syncthreads();
    pipe.convert_s(0);
    load_s(1, 0);
    const bool two = np > 32;
    for (int t = 0; t < n_steps; ++t) {
        pipe.load_c(min(t + 1, n_steps - 1));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            pipe.convert_s(1 - h);
            pipe.products(lds.C[t & 1], h, 0, accr[0], acci[0]);
            pipe.pin(1 - h);
            load_s(h == 0 ? t + 1 : t + 2, 1 - h);
            __builtin_amdgcn_sched_barrier(0);
            if (two) pipe.products(lds.C[t & 1], h, 1, accr[1], acci[1]);
        }
        pipe.stage_c(lds.C[(t + 1) & 1]);
        const int4 s = step[t];
        if (__builtin_amdgcn_readfirstlane(s.w)) {
            const int k = __builtin_amdgcn_readfirstlane(s.z);
            float2* out = a.T + ((size_t)k * ns + py) * a.n_cols * m;
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    if (sum_row(rb, r, 0) >= np) continue;        // no rows left here (uniform)
                    const int row = sum_row(rb, r, half), q = lds.idx[row];
                    const int u = (px - lds.at[row].x) & (ns - 1);
                    if (q >= 0 && u < m) out[(size_t)q * m + u] = make_float2(accr[rb][0][r], acci[rb][0][r]);
                }
            clear(accr);
            clear(acci);
        }
        __syncthreads();
    }
}

// Windows of up to 64 probes of one scan column on 128 pixels of T (1, 2, 4 or
// 8 rows of the S grid).  T is FP32, and so are these products.
__global__ __launch_bounds__(mfmac::NT) __attribute__((amdgpu_waves_per_eu(3))) void k_sum_ky(TwoStage a) {
    using namespace mfmac;
    __shared__ ContractLds<3> lds;
    int l = (blockIdx.x & 7) * a.per_xcd + (blockIdx.x >> 3);
    if (l >= a.n_blocks) return;
    const int ns = a.ns, m = a.m, w = min(m, 128), R = 128 / w, nu = m / w;
    const int chunk = l % a.chunks;
    l /= a.chunks;
    const int ut = l % nu;
    l /= nu;
    const int y0 = l % (ns / R) * R, q = l / (ns / R);
    const int e0 = a.col_start[q], n = a.col_start[q + 1] - e0;
    int first, count;
    cover_run(a.entry_corner + e0, n, y0, R, m, ns, first, count);
    const int np = min(PC, count - chunk * PC);
    if (np <= 0) return;
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, half = lane >> 5;
    if (tid < PC) {
        const int e = e0 + (first + chunk * PC + tid) % n;
        lds.idx[tid] = tid < np ? a.entry_probe[e] : -1;
        lds.at[tid] = make_int2(0, tid < np ? a.entry_corner[e] : 0);
    }
    __syncthreads();
    const int at = (tid >> 6) * 32 + col, py = y0 + at / w, u = ut * 128 + at % w;
    const int pix[1] = {(at / w) * a.n_cols * m + u};
    Sums<1> sum;
    sum_beams<3, 1, 1 << 30>(lds, a.T + ((size_t)y0 * a.n_cols + q) * m, (size_t)ns * a.n_cols * m, a.n_rows, pix, a.cy,
                 (a.n_rows + KSTEP - 1) / KSTEP, np > 32, sum);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = sum_row(rb, r, half), p = lds.idx[row];
            const int v = (py - lds.at[row].y) & (ns - 1);
            if (p >= 0 && v < m)
                a.win[(size_t)p * m * m + (size_t)v * m + u] = make_float2(sum.r[rb][0][r], sum.i[rb][0][r]);
        }
}

// C operands of both stages, FP32.  Columns: coefficients at (x, 0) over the K
// steps; probes: e^{-2 pi i ky y / L} over ky.
__global__ __launch_bounds__(WG) void k_two_stage_operands(u32x4* __restrict__ cx, u32x4* __restrict__ cy,
                                                           const double2* __restrict__ col_xy,
                                                           const double2* __restrict__ xy, const int2* __restrict__ beams,
                                                           const float2* __restrict__ aberr,
                                                           const int4* __restrict__ steps,
                                                           const int4* __restrict__ rows, int n_cols, int col_steps,
                                                           int n_probes, int n_rows, double inv_L, float amp) {
    const int K2 = (n_rows + KSTEP - 1) / KSTEP;
    const int64_t nx = (int64_t)n_cols * col_steps * 4, total = nx + (int64_t)n_probes * K2 * 4;
    for (int64_t i = (int64_t)blockIdx.x * WG + threadIdx.x; i < total; i += (int64_t)gridDim.x * WG) {
        float2 v[4];
        if (i < nx) {
            const int q = (int)((i >> 2) / col_steps), k = (int)((i >> 2) % col_steps), g = (int)(i & 3);
            const int4 step = steps[k];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                v[j] = g * 4 + j < step.y ? coefficient(col_xy[q], beams[step.x + g * 4 + j], aberr, step.x + g * 4 + j, inv_L, amp)
                                          : make_float2(0.f, 0.f);
            store_operand<3>(cx + (i >> 2) * REC<3>, g, v);
        } else {
            const int64_t o = i - nx;
            const int p = (int)((o >> 2) / K2), k = (int)((o >> 2) % K2), g = (int)(o & 3);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = k * KSTEP + g * 4 + j;
                v[j] = r < n_rows ? coefficient(xy[p], make_int2(0, rows[r].w), nullptr, 0, inv_L, 1.f) : make_float2(0.f, 0.f);
            }
            store_operand<3>(cy + (o >> 2) * REC<3>, g, v);
        }
    }
}

hipError_t launch_two_stage_operands(const TwoStageArgs& t, hipStream_t st) {
    const int K2 = ksteps_of(t.n_rows);
    const int64_t total = ((int64_t)t.n_cols * t.col_steps + (int64_t)t.n_probes * K2) * 4;
    const int64_t blocks = std::min<int64_t>((total + WG - 1) / WG, 65536);
    hipLaunchKernelGGL(k_two_stage_operands, dim3((unsigned)blocks), dim3(WG), 0, st, static_cast<u32x4*>(t.cx),
                       static_cast<u32x4*>(t.cy), t.col_xy, t.xy, t.beams, t.aberr, t.steps, t.rows, t.n_cols,
                       t.col_steps, t.n_probes, t.n_rows, t.inv_L, t.amp);
    return hipGetLastError();
}

size_t two_stage_cx_bytes(int n_cols, int col_steps) { return (size_t)n_cols * col_steps * 16 * REC<3>; }
size_t two_stage_cy_bytes(int64_t n_probes, int n_rows) { return (size_t)n_probes * ksteps_of(n_rows) * 16 * REC<3>; }
size_t two_stage_column_bytes(int n_rows, int ns, int m) { return (size_t)n_rows * ns * m * sizeof(float2); }

int two_stage_columns(const TwoStageArgs& t) {
    return two_stage_columns_per_launch(t.n_cols, t.n_rows, t.ns, t.m, t.T_bytes);
}

static TwoStage two_stage_launch(const TwoStageArgs& t, int q0, int n) {
    TwoStage a{};
    a.S = t.S;
    a.T = t.T;
    a.win = t.win;
    a.cx = static_cast<const u32x4*>(t.cx) + (size_t)q0 * t.col_steps * REC<3>;
    a.cy = static_cast<const u32x4*>(t.cy);
    a.rows = t.rows;
    a.steps = t.steps;
    a.col_corner = t.col_corner + q0;
    a.col_start = t.col_start + q0;
    a.entry_corner = t.entry_corner;
    a.entry_probe = t.entry_probe;
    a.n_cols = n;
    a.n_rows = t.n_rows;
    a.col_steps = t.col_steps;
    a.ns = t.ns;
    a.m = t.m;
    a.tile_width = t.tile_width;
    return a;
}
static hipError_t start_two_stage(void (*kernel)(TwoStage), TwoStage& a, int64_t blocks, hipStream_t st) {
    if (!launchable(blocks)) return hipErrorInvalidValue;
    a.n_blocks = (int)blocks;
    a.per_xcd = (a.n_blocks + 7) / 8;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(8 * a.per_xcd)), dim3(mfmac::NT), 0, st, a);
    return hipGetLastError();
}

int64_t two_stage_blocks(const TwoStageArgs& t) {
    const int64_t tiles = sum_kx_tiles(t.ns, t.max_cols);
    const int64_t kx = tiles * sum_kx_row_groups(tiles, t.n_rows, ksteps_of(t.max_row_beams), MAX_STEPS);
    const int64_t ky = sum_ky_blocks(two_stage_columns(t), t.ns, t.m, t.max_probes);
    return launchable(kx) && launchable(ky) ? kx + ky : -1;
}

hipError_t launch_sum_kx(int precision, const TwoStageArgs& t, int q0, int n, hipStream_t st) {
    TwoStage a = two_stage_launch(t, q0, n);
    a.chunks = (t.max_cols + mfmac::PC - 1) / mfmac::PC;
    const int64_t tiles = sum_kx_tiles(t.ns, t.max_cols);
    a.row_groups = sum_kx_row_groups(tiles, t.n_rows, ksteps_of(t.max_row_beams), MAX_STEPS);
    return start_two_stage(precision == 0 ? k_sum_kx<3> : k_sum_kx<2>, a, tiles * a.row_groups, st);
}

hipError_t launch_sum_ky(const TwoStageArgs& t, int q0, int n, hipStream_t st) {
    if (n > two_stage_columns(t)) return hipErrorInvalidValue;
    TwoStage a = two_stage_launch(t, q0, n);
    a.chunks = (t.max_probes + mfmac::PC - 1) / mfmac::PC;
    return start_two_stage(k_sum_ky, a, sum_ky_blocks(n, t.ns, t.m, t.max_probes), st);
}

// ------------------------------------------------ deterministic bin sums --
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// ------------------------------------------------------- window detection --
// One workgroup per probe: row transforms, M x M window in LDS, column
// transforms, |Psi|^2 / M^4, then each bin summed over its pixel list.
struct WindowJob {
    const float2* win;        // [n_probes][m][m]
    float* out;               // [n_probes][n_bins], or null
    float* diff;              // [n_probes][m][m] intensities (4D output), or null
    const int* perm;          // window pixels grouped by bin
    const int* bin_start;     // [n_bins + 1]
    const float2* tw_m;       // W_m twiddles
    int n_bins;
    int probe0;               // first probe of this job among those of the launch
    float scale;              // out = scale * sum (+ out when accumulating)
    int accumulate;
};
struct WindowBatch {
    int n_jobs;
    int n_probes;             // over all jobs
    WindowJob job[MAX_JOBS];
};

// Rows go straight from memory to their transform's registers and stay there;
// LDS holds one plane of floats, M + M / 8 or M + M / 16 square, through which
// real parts and then imaginary parts pass: the exchanges of the row transforms
// (each in the padded slots of its own row), the transposition, the exchanges of
// the column transforms (each in its own column), and last the intensities,
// which are summed into bins by BL lanes each.
//
// Bound: LDS and latency.  Half the LDS of complex values gives a 128-point
// window two workgroups per CU instead of one.  The row stride of 8 modulo 64
// (M = 64 and 128) spreads rows and columns over all banks; conflicts take a
// fifth of the active cycles at 128.
// 16,384 probes of 128^2: 1.30 (complex window, the next rows loaded beside the
// columns) -> 0.64 ms; 16,384 of 64^2: 216 -> 160 us; 256 of 64^2: 8.6 us either
// way.  128-point transforms are 16 x 8 points (one exchange).  Lanes per bin at
// 128: 16 and 32 within 2%, 64 0.15 ms slower; a wavefront per bin took 16 us
// more for 256 windows of 64^2.
template <int M> struct WinFft { using type = Fft<M>; };
template <> struct WinFft<128> { using type = FftT<128, PlanWin128>; };
template <int M>
struct WinCfg {
    using F = typename WinFft<M>::type;
    static constexpr int NW = M >= 64 ? 8 : 4;                // wavefronts per workgroup
    static constexpr int BL = M >= 128 ? 16 : 8;              // lanes per bin
    static constexpr int NT = 64 * NW;
};

// Job of probe p of a launch, copied out by value (see locate).
__device__ __forceinline__ WindowJob window_job(const WindowBatch& batch, int p) {
    int jj = 0;
#pragma unroll
    for (int k = 1; k < MAX_JOBS; ++k)
        if (k < batch.n_jobs && batch.job[k].probe0 <= p) jj = k;
    return batch.job[jj];
}

template <int M>
__global__ __launch_bounds__(WinCfg<M>::NT) __attribute__((amdgpu_waves_per_eu(4))) void k_window_detect(WindowBatch batch) {
    using C = WinCfg<M>;
    using F = typename C::F;
    constexpr int E = F::E, LPT = F::LPT, G = 64 / LPT, NT = C::NT, RS = F::LDS, BL = C::BL;
    constexpr int STEP = C::NW * G, NR = (M + STEP - 1) / STEP;   // rows (and columns) r0 + i STEP of a lane
    __shared__ float buf[RS * RS];
    const int tid = threadIdx.x, lane = tid & 63, lt = lane % LPT;
    const int r0 = (tid >> 6) * G + lane / LPT;
    const WindowJob job = window_job(batch, blockIdx.x);
    const int p = (int)blockIdx.x - job.probe0, n_bins = job.n_bins;
    float2 v[NR][E];
    const float2* w = job.win + (size_t)p * M * M;
#pragma unroll
    for (int i = 0; i < NR; ++i)
        if (r0 + i * STEP < M)
#pragma unroll
            for (int e = 0; e < E; ++e) v[i][e] = w[(r0 + i * STEP) * M + lt + LPT * e];
    typename F::Twiddles tw;
    tw.load(job.tw_m, lt);
#pragma unroll
    for (int i = 0; i < NR; ++i)
        if (r0 + i * STEP < M)
            F::template run_x<-1>(v[i], typename F::template PlaneX<1>{buf + (r0 + i * STEP) * RS}, tw, lt);
    auto transpose = [&](float float2::*part) {
        F::sync();
#pragma unroll
        for (int i = 0; i < NR; ++i)
            if (r0 + i * STEP < M)
#pragma unroll
                for (int e = 0; e < E; ++e) buf[(r0 + i * STEP) * RS + lt + LPT * e] = v[i][e].*part;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NR; ++i)
            if (r0 + i * STEP < M)
#pragma unroll
                for (int e = 0; e < E; ++e) v[i][e].*part = buf[(lt + LPT * e) * RS + r0 + i * STEP];
    };
    transpose(&float2::x);
    __syncthreads();                                          // the imaginary parts overwrite the real ones
    transpose(&float2::y);
    // from here a lane's transforms touch their own columns only
    const float scale = 1.0f / ((float)M * (float)M * (float)M * (float)M);
#pragma unroll
    for (int i = 0; i < NR; ++i)
        if (r0 + i * STEP < M) {
            float* col = buf + r0 + i * STEP;
            F::template run_x<-1>(v[i], typename F::template PlaneX<RS>{col}, tw, lt);
            F::sync();
#pragma unroll
            for (int e = 0; e < E; ++e) col[(lt + LPT * e) * RS] = cnorm(v[i][e]) * scale;
        }
    __syncthreads();
    if (job.diff) {
        // the 4D output takes the same scale and accumulation as the 3D one
        float* d = job.diff + (size_t)p * M * M;
        for (int idx = tid; idx < M * M; idx += NT) {
            const float s = job.scale * buf[(idx / M) * RS + idx % M];
            d[idx] = job.accumulate ? d[idx] + s : s;
        }
    }
    if (job.out)
        for (int b = tid / BL; b < n_bins; b += NT / BL) {
            float s = 0.f;
            const int k1 = job.bin_start[b + 1];
#pragma unroll 4
            for (int k = job.bin_start[b] + tid % BL; k < k1; k += BL) {
                const int pix = job.perm[k];
                s += buf[(pix / M) * RS + pix % M];
            }
#pragma unroll
            for (int off = BL / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, BL);
            if (tid % BL == 0) {
                float* o = job.out + (size_t)p * n_bins + b;
                *o = job.accumulate ? *o + job.scale * s : job.scale * s;
            }
        }
}

template <int M>
static hipError_t window_m(const WindowArgs* jobs, int n_jobs, hipStream_t st) {
    for (int j0 = 0; j0 < n_jobs; j0 += MAX_JOBS) {
        WindowBatch b{};
        b.n_jobs = n_jobs - j0 < MAX_JOBS ? n_jobs - j0 : MAX_JOBS;
        for (int k = 0; k < b.n_jobs; ++k) {
            const WindowArgs& a = jobs[j0 + k];
            b.job[k] = WindowJob{a.win, a.out, a.diff, a.perm, a.bin_start, a.tw_m, a.n_bins, b.n_probes, a.scale,
                                 a.accumulate};
            b.n_probes += a.n_probes;
        }
        if (b.n_probes == 0) continue;
        hipLaunchKernelGGL((k_window_detect<M>), dim3((unsigned)b.n_probes), dim3(WinCfg<M>::NT), 0, st, b);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------- large windows (M = 256, 512) --
// A window no longer fits in LDS: rows are transformed in place in HBM, then
// 16-column strips are staged through LDS for the column transforms, which
// write |Psi|^2 / M^4 to an intensity buffer binned by k_bin_reduce.
template <int M>
__global__ __launch_bounds__(WG) void k_window_rows(float2* __restrict__ win, const float2* __restrict__ tw_m,
                                                    int64_t n_rows) {
    using F = Fft<M>;
    constexpr int E = F::E, LPT = F::LPT, G = 64 / LPT;
    __shared__ float2 xch[4 * G * F::LDS];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int g = lane / LPT, lt = lane % LPT;
    const int64_t r = (int64_t)blockIdx.x * 4 * G + wave * G + g;
    if (r >= n_rows) return;
    typename F::Twiddles tw;
    tw.load(tw_m, lt);
    float2* row = win + r * M;
    float2 v[E];
#pragma unroll
    for (int i = 0; i < E; ++i) v[i] = row[lt + LPT * i];
    F::template run<-1>(v, xch + (wave * G + g) * F::LDS, tw, lt);
#pragma unroll
    for (int i = 0; i < E; ++i) row[lt + LPT * i] = v[i];
}

template <int M>
__global__ __launch_bounds__(WG) void k_window_cols(const float2* __restrict__ win, float* __restrict__ inten,
                                                    const float2* __restrict__ tw_m) {
    using F = Fft<M>;
    constexpr int E = F::E, LPT = F::LPT, G = 64 / LPT, CW = 16, ROWS = CW + 1;
    __shared__ float2 strip[M * ROWS];
    __shared__ float2 xch[4 * G * F::LDS];
    const int p = blockIdx.y, u0 = blockIdx.x * CW;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int g = lane / LPT, lt = lane % LPT;
    const float2* w = win + (size_t)p * M * M;
    {
        constexpr int NLD = M * CW / WG;
        float2 ld[NLD];
#pragma unroll
        for (int k = 0; k < NLD; ++k) {
            const int idx = tid + k * WG, v = idx / CW, c = idx % CW;
            ld[k] = w[(size_t)v * M + u0 + c];
        }
#pragma unroll
        for (int k = 0; k < NLD; ++k) {
            const int idx = tid + k * WG, v = idx / CW, c = idx % CW;
            strip[v * ROWS + c] = ld[k];
        }
    }
    __syncthreads();
    typename F::Twiddles tw;
    tw.load(tw_m, lt);
    const float scale = 1.0f / ((float)M * (float)M * (float)M * (float)M);
    float* I = inten + (size_t)p * M * M;
    for (int c0 = wave * G; c0 < CW; c0 += 4 * G) {
        const int c = c0 + g;
        float2* col = strip + c;
        float2 v[E];
#pragma unroll
        for (int i = 0; i < E; ++i) v[i] = col[(lt + LPT * i) * ROWS];
        F::template run<-1>(v, xch + (wave * G + g) * F::LDS, tw, lt);
#pragma unroll
        for (int i = 0; i < E; ++i) I[(size_t)(lt + LPT * i) * M + u0 + c] = cnorm(v[i]) * scale;
    }
}

// diff = scale * inten (+ diff when accumulating): the 4D output of a large
// window when it is scaled or accumulated (the bins read the plain intensity).
__global__ __launch_bounds__(WG) void k_scale_into(float* __restrict__ diff, const float* __restrict__ inten,
                                                   int64_t count, float scale, int accumulate) {
    for (int64_t i = (int64_t)blockIdx.x * WG + threadIdx.x; i < count; i += (int64_t)gridDim.x * WG) {
        const float v = scale * inten[i];
        diff[i] = accumulate ? diff[i] + v : v;
    }
}

template <int M>
static hipError_t window_large(float2* win, float* inten, float* out, const int* perm, const int* bin_start,
                               const float2* tw_m, int n_probes, int n_bins, float scale, int accumulate,
                               hipStream_t st) {
    // inten receives |Psi|^2 / M^4 (it is the 4D output when one is requested
    // unscaled and not accumulated)
    constexpr int G = 64 / Fft<M>::LPT;
    const int64_t rows = (int64_t)n_probes * M;
    hipLaunchKernelGGL((k_window_rows<M>), dim3((unsigned)((rows + 4 * G - 1) / (4 * G))), dim3(WG), 0, st, win,
                       tw_m, rows);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_window_cols<M>), dim3(M / 16, (unsigned)n_probes), dim3(WG), 0, st, win, inten, tw_m);
    e = hipGetLastError();
    if (e != hipSuccess || !out) return e;
    return launch_bin_reduce(inten, (int64_t)M * M, out, perm, bin_start, n_probes, n_bins, st, scale, accumulate);
}

hipError_t launch_window_batch(int m, const WindowArgs* jobs, int n_jobs, hipStream_t st) {
    switch (m) {
        case 16: return window_m<16>(jobs, n_jobs, st);
        case 32: return window_m<32>(jobs, n_jobs, st);
        case 64: return window_m<64>(jobs, n_jobs, st);
        case 128: return window_m<128>(jobs, n_jobs, st);
        case 256:
        case 512:
            for (int k = 0; k < n_jobs; ++k) {
                const WindowArgs& a = jobs[k];
                const bool direct = a.diff && a.scale == 1.0f && !a.accumulate;
                float* I = direct ? a.diff : a.inten;
                hipError_t e = m == 256 ? window_large<256>(a.win, I, a.out, a.perm, a.bin_start, a.tw_m,
                                                            a.n_probes, a.n_bins, a.scale, a.accumulate, st)
                                        : window_large<512>(a.win, I, a.out, a.perm, a.bin_start, a.tw_m,
                                                            a.n_probes, a.n_bins, a.scale, a.accumulate, st);
                if (e != hipSuccess) return e;
                if (a.diff && !direct) {
                    const int64_t count = (int64_t)a.n_probes * m * m;
                    const int64_t blocks = std::min<int64_t>((count + WG - 1) / WG, 65536);
                    hipLaunchKernelGGL(k_scale_into, dim3((unsigned)blocks), dim3(WG), 0, st, a.diff, a.inten, count,
                                       a.scale, a.accumulate);
                    e = hipGetLastError();
                    if (e != hipSuccess) return e;
                }
            }
            return hipSuccess;
    }
    return hipErrorInvalidValue;
}

// ------------------------------------------------------------- bin reduce --
// One wavefront per (item, bin).  Bound: latency of the gathered loads, several
// of which are in flight at once.  64 items, 62 bins of a 512^2 band: 418 -> 30
// us; 134 bins of a 128^2 band: 42 -> 7.5 us, against one workgroup per item
// that took its bins in turn.
__global__ __launch_bounds__(WG) void k_bin_reduce(const float* __restrict__ inten, int64_t pix_per_item,
                                                   float* __restrict__ out, const int* __restrict__ perm,
                                                   const int* __restrict__ bin_start, int n_bins, int groups,
                                                   float scale, int accumulate) {
    const int item = blockIdx.x / groups, lane = threadIdx.x & 63;
    const float* I = inten + (size_t)item * pix_per_item;
    for (int64_t b = blockIdx.x % groups * 4 + (threadIdx.x >> 6); b < n_bins; b += 4 * groups) {
        const int k1 = bin_start[b + 1];
        float s = 0.f;
#pragma unroll 8
        for (int k = bin_start[b] + lane; k < k1; k += 64) s += I[perm[k]];
        s = wave_sum(s);
        if (lane == 0) {
            float* o = out + (size_t)item * n_bins + b;
            *o = accumulate ? *o + scale * s : scale * s;
        }
    }
}

hipError_t launch_bin_reduce(const float* inten, int64_t pix_per_item, float* out, const int* perm,
                             const int* bin_start, int n_items, int n_bins, hipStream_t st, float scale,
                             int accumulate) {
    const int groups = bin_groups(n_bins), most = bin_items(n_bins);
    for (int64_t i = 0; i < n_items; i += most) {
        const int n = (int)std::min<int64_t>(most, n_items - i);
        hipLaunchKernelGGL(k_bin_reduce, dim3((unsigned)n * groups), dim3(WG), 0, st, inten + (size_t)i * pix_per_item,
                           pix_per_item, out + (size_t)i * n_bins, perm, bin_start, n_bins, groups, scale, accumulate);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace prism
