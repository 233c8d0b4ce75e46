// probe.hip -- PRISM probe synthesis: coefficients, windowed beam contraction,
// window FFT with |Psi|^2, and deterministic annular-detector sums.
//
// "PRISM Probe Simulations": each probe is a sum over plane waves of the
// cropped S-matrix layers times per-beam phase coefficients; the modulus
// squared of the FFT of that exit wave is binned into detectors (Fig. 1i-k).
#include "fft.hpp"
#include "kernels.hpp"

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
    const float2* S;          // S-matrix: complex64 [n_beams][ns][ns]
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
//                   left out (ml, lm, ll) is at most 2^-25 of the product,
//                   below the rounding of an FP32 product.
//   NP = 2 (split)  16 bits; hh, hl, lh (lo lo, ~2^-16 relative, left out).
//   NP = 1 (BF16)   hh.
//
// A workgroup is one work tile (FP32: half of one) x PC = 64 probes: a wave
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
// probes of 256^2 windows: 1.16 + 1.07 -> 1.02 ms).  FP32 products on the
// VALU: 2025 probes x 1245 beams x 128^2, 7.1 -> 2.0 ms with six BF16 products.
namespace mfmac {
constexpr int NT = 256;               // threads per workgroup
constexpr int PC = 64;                // probes per workgroup
constexpr int RB = PC / 32;           // 32-probe row blocks
constexpr int SUB = 8;                // beams per MFMA step, half a K step
// 32-pixel column blocks (pairs of tile rows) per wave.  FP32 takes one, and
// two workgroups per tile, so that the registers of the other hold the sum
// of the last FLUSH K steps apart from the running total: an FP32 sum of
// 1245 beams, 6 products each, is otherwise rounded 936 times at the size of
// the total (2025 probes of 1245 beams: error against 64 bits 1.4e-7 on the
// VALU, 1.7e-7 without the split total, 9e-8 with it).
template <int NP> constexpr int CBS = NP == 3 ? 1 : 2;
template <int NP> constexpr int SPLITS = 2 / CBS<NP>;   // workgroups per (tile, probe chunk)
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

// C operands, thread = (probe, group of 4 beams): split records
// [probe][K step][part][4-beam group] for NP = 1, 2, and the FP32 values
// [probe][K step][16 beams] (the same bytes as NP = 2) for NP = 3, which the
// contraction splits as it stages them.  Beams past the last are zero.
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
        if constexpr (NP == 3) {
            float4* dst = reinterpret_cast<float4*>(C) + i * 2;
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
            u32x4* rec = C + ((size_t)p * K + k) * NP * 4;
#pragma unroll
            for (int part = 0; part < NP; ++part) rec[part * 4 + g] = ch[part];
        }
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

template <int NP>
__global__ __launch_bounds__(mfmac::NT) __attribute__((amdgpu_waves_per_eu(2))) void k_contract(ContractBatch batch) {
    using namespace mfmac;
    constexpr int CB = CBS<NP>;
    constexpr int NCH = NP * 4;                   // 16-byte chunks per record
    // probe stride of an LDS chunk row: odd (or = 2 mod 8 when 4 lanes write
    // one probe) so that 8 lanes of a staging store hit distinct bank groups
    constexpr int LP = NP == 3 ? PC + 2 : PC + 1;
    __shared__ u32x4 Cl[2][NCH * LP];
    __shared__ int pidx[PC];
    __shared__ int2 pcorner[PC];

    int tile, chunk;
    ContractJob job;
    if (!locate(batch, job, tile, chunk)) return;
    const int row0 = 8 * CB * (chunk % SPLITS<NP>);   // first tile row of this workgroup
    chunk /= SPLITS<NP>;
    float2* __restrict__ win = job.win;
    const int ns = job.ns, m = job.m, K = job.ksteps, n_beams = job.n_beams;
    const int t0 = job.tile_start[tile], t1 = job.tile_start[tile + 1];
    const int pc0 = t0 + chunk * PC;
    if (pc0 >= t1) return;
    const int np = min(PC, t1 - pc0);
    const int2 org = job.tile_origin[tile];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int col = lane & 31, half = lane >> 5;
    if (tid < PC) {
        const int q = tid < np ? job.tile_probes[pc0 + tid] : -1;
        pidx[tid] = q;
        pcorner[tid] = q >= 0 ? job.corner[q] : make_int2(0, 0);
    }
    __syncthreads();

    f32x16 accr[RB][CB], acci[RB][CB];
#pragma unroll
    for (int a = 0; a < RB; ++a)
#pragma unroll
        for (int b = 0; b < CB; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) accr[a][b][r] = acci[a][b][r] = 0.f;
    f32x16 totr[RB][CB], toti[RB][CB];            // running totals (NP = 3)
    if constexpr (NP == 3) {
#pragma unroll
        for (int a = 0; a < RB; ++a)
#pragma unroll
            for (int b = 0; b < CB; ++b) {
                totr[a][b] = accr[a][b];
                toti[a][b] = acci[a][b];
            }
    }

    // S operand of this lane: pixel (py, px) of column block cb; byte offsets
    // from the start of the step, read by buffer loads from a scalar resource
    // that ends with the last beam, so that beams past it read as zero and
    // the loop holds no branch around a load (each would end in a wait for
    // all loads in flight)
    const size_t plane = (size_t)ns * ns;
    const int plane_bytes = (int)(plane * sizeof(float2));
    int voff[CB][4];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
        const int py = (org.y + row0 + 2 * (CB * wave + cb) + (col >> 4)) & (ns - 1), px = (org.x + (col & 15)) & (ns - 1);
#pragma unroll
        for (int j = 0; j < 4; ++j) voff[cb][j] = (py * ns + px) * (int)sizeof(float2) + (4 * half + j) * plane_bytes;
    }
    float2 raw[2][CB][4];
    auto load_s = [&](int k, int h) {
        const int b0 = min(k * KSTEP + h * SUB, n_beams);
        const int64_t left = (int64_t)(n_beams - b0) * plane_bytes;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float2*>(job.S + (size_t)b0 * plane), (short)0,
            (int)min(left, (int64_t)0x7fffffff), 0x00020000);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                raw[h][cb][j] = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rs, voff[cb][j], 0, 0));
    };
    // C staging.  NP <= 2: chunk (tid + j NT) of the K step's PC records;
    // NP = 3: the 4 beams (tid % 4) of probe tid / 4, split when stored.
    // Rows past np read probe 0's record; they are not stored.
    constexpr int CW = NP == 3 ? 2 : NP, NCP = NP == 3 ? 1 : NP;
    u32x4 creg[CW];
    const u32x4* cptr[NCP];
#pragma unroll
    for (int j = 0; j < NCP; ++j) {
        const int q = max(pidx[NP == 3 ? tid / 4 : (tid + j * NT) / NCH], 0);
        const int off = NP == 3 ? (tid % 4) * 2 : (tid + j * NT) % NCH;
        cptr[j] = static_cast<const u32x4*>(job.C) + (size_t)q * K * (NP == 3 ? 8 : NCH) + off;
    }
    auto load_c = [&](int k) {
        const size_t at = (size_t)min(k, K - 1) * (NP == 3 ? 8 : NCH);
#pragma unroll
        for (int j = 0; j < CW; ++j) creg[j] = NP == 3 ? cptr[0][at + j] : cptr[NP == 3 ? 0 : j][at];
    };
    auto stage_c = [&](u32x4* dst) {
        if constexpr (NP == 3) {
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
    };
    // B operands of the two steps of a K step: step s + 1 is converted while
    // the products of step s run
    u32x4 B[2][NP][CB];
    auto convert_s = [&](int h) {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                unsigned int w[NP];
                split_parts<NP>(raw[h][cb][j].x, raw[h][cb][j].y, w);
#pragma unroll
                for (int part = 0; part < NP; ++part) B[h][part][cb][j] = w[part];
            }
    };
    load_c(0);
    load_s(0, 0);
    load_s(0, 1);
    stage_c(Cl[0]);
    __syncthreads();
    convert_s(0);
    load_s(1, 0);

    const bool two = np > 32;                     // the second row block holds probes
    for (int k0 = 0; k0 < K; k0 += FLUSH<NP>) {
        const int k1 = min(k0 + FLUSH<NP>, K);
        for (int k = k0; k < k1; ++k) {
            const u32x4* Ck = Cl[k & 1];
            load_c(k + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                convert_s(1 - h);
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    if (rb > 0 && !two) break;
                    u32x4 A[NP];
#pragma unroll
                    for (int part = 0; part < NP; ++part) A[part] = Ck[(part * 4 + 2 * h + half) * LP + 32 * rb + col];
                    auto product = [&](f32x16 (&acc)[CB], int pa, int pb) {
#pragma unroll
                        for (int cb = 0; cb < CB; ++cb)
                            acc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(A[pa]), as_bf16x8(B[h][pb][cb]),
                                                                              acc[cb], 0, 0, 0);
                    };
                    auto products = [&](f32x16 (&acc)[CB]) {
                        if constexpr (NP == 3) {
                            product(acc, 2, 0);
                            product(acc, 0, 2);
                            product(acc, 1, 1);
                        }
                        if constexpr (NP >= 2) {
                            product(acc, 1, 0);
                            product(acc, 0, 1);
                        }
                        product(acc, 0, 0);
                    };
#pragma unroll
                    for (int part = 0; part < NP; ++part) A[part] ^= 0x80000000u;             // (Cr, -Ci)
                    products(accr[rb]);
#pragma unroll
                    for (int part = 0; part < NP; ++part) {                                   // (Ci, Cr)
                        A[part] ^= 0x80000000u;
                        A[part] = (A[part] >> 16) | (A[part] << 16);
                    }
                    products(acci[rb]);
                    if (rb == 0) {
                        // the loads reuse the registers that the conversion
                        // frees: it ends here (not sunk to where its results
                        // are used), and the loads are not moved down
#pragma unroll
                        for (int part = 0; part < NP; ++part)
#pragma unroll
                            for (int cb = 0; cb < CB; ++cb) asm volatile("" : "+v"(B[1 - h][part][cb]));
                        __builtin_amdgcn_sched_barrier(0);
                        load_s(h == 0 ? k + 1 : k + 2, 1 - h);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
            stage_c(Cl[(k + 1) & 1]);
            __syncthreads();
        }
        if constexpr (NP == 3) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) {
                    totr[rb][cb] += accr[rb][cb];
                    toti[rb][cb] += acci[rb][cb];
#pragma unroll
                    for (int r = 0; r < 16; ++r) accr[rb][cb][r] = acci[rb][cb][r] = 0.f;
                }
        }
    }
    // ---- epilogue: D register r = probe row (r & 3) + 8 (r >> 2) + 4 half, column = pixel
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = 32 * rb + (r & 3) + 8 * (r >> 2) + 4 * half;
            const int q = pidx[row];
            if (q < 0) continue;
            const int2 c0 = pcorner[row];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                const int py = org.y + row0 + 2 * (CB * wave + cb) + (col >> 4), px = org.x + (col & 15);
                const int v = (py - c0.y) & (ns - 1);
                const int u = (px - c0.x) & (ns - 1);
                if (v < m && u < m) {
                    float2* w = win + (size_t)q * m * m + (size_t)v * m + u;
                    float2 res = NP == 3 ? make_float2(totr[rb][cb][r], toti[rb][cb][r]) : make_float2(accr[rb][cb][r], acci[rb][cb][r]);
                    if (job.accumulate) res = cadd(*w, res);
                    *w = res;
                }
            }
        }
}

int contract_probe_chunk() { return mfmac::PC; }

hipError_t launch_contract_batch(int precision, const ContractArgs* jobs, int n_jobs, hipStream_t st) {
    for (int j0 = 0; j0 < n_jobs; j0 += MAX_JOBS) {
        ContractBatch b{};
        b.n_jobs = n_jobs - j0 < MAX_JOBS ? n_jobs - j0 : MAX_JOBS;
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
            job.chunks = std::max(1, (a.max_per_tile + mfmac::PC - 1) / mfmac::PC) *
                         (precision == 0 ? mfmac::SPLITS<3> : mfmac::SPLITS<2>);
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
            launch(k_contract<3>);
        else if (precision == 1)
            launch(k_contract<2>);
        else
            launch(k_contract<1>);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ------------------------------------------------ deterministic bin sums --
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// ------------------------------------------------------- window detection --
// One workgroup per probe: M x M window in LDS, row then column transforms,
// |Psi|^2 / M^4, then each bin summed over its pixel list by one wavefront.
struct WindowJob {
    const float2* win;        // [n_probes][m][m]
    float* out;               // [n_probes][n_bins], or null
    float* diff;              // [n_probes][m][m] intensities (4D output), or null
    const int* perm;          // window pixels grouped by bin
    const int* bin_start;     // [n_bins + 1]
    const float2* tw_m;       // W_m twiddles
    int n_bins;
    int probe0;               // first workgroup of this job
    float scale;              // out = scale * sum (+ out when accumulating)
    int accumulate;
};
struct WindowBatch {
    int n_jobs;
    WindowJob job[MAX_JOBS];
};

// The window sits in LDS with an odd row stride RS of at least the padded
// exchange length and with that many rows (more than M), so that each row
// transform and each column transform exchanges in place, through the
// padded slots of its own row or column: no separate exchange buffers, so
// the 128-point windows take 16 wavefronts per workgroup in the LDS that
// would otherwise hold 4 wavefronts' exchange buffers.  The odd stride keeps
// the strided column accesses of 16 lanes in distinct banks.
template <int M>
struct WinCfg {
    using F = Fft<M>;
    static constexpr int NW = M >= 128 ? 16 : 4;              // wavefronts per workgroup
    static constexpr int NT = 64 * NW;
    static constexpr int RS = F::LDS | 1;                     // row stride (float2), odd
    static constexpr int ROWS = F::LDS;                       // rows (the column exchanges use all)
};

template <int M>
__global__ __launch_bounds__(WinCfg<M>::NT) void k_window_detect(WindowBatch batch) {
    using C = WinCfg<M>;
    using F = typename C::F;
    constexpr int E = F::E, LPT = F::LPT, G = 64 / LPT, NW = C::NW, NT = C::NT, RS = C::RS;
    __shared__ float2 buf[C::ROWS * RS];
    int jj = 0;
#pragma unroll
    for (int k = 1; k < MAX_JOBS; ++k)
        if (k < batch.n_jobs && batch.job[k].probe0 <= (int)blockIdx.x) jj = k;
    const WindowJob job = batch.job[jj];
    const float2* __restrict__ win = job.win;
    float* __restrict__ out = job.out;
    float* __restrict__ diff = job.diff;
    const int* __restrict__ perm = job.perm;
    const int* __restrict__ bin_start = job.bin_start;
    const float2* __restrict__ tw_m = job.tw_m;
    const int n_bins = job.n_bins;
    const int p = (int)blockIdx.x - job.probe0;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int g = lane / LPT, lt = lane % LPT;
    const float2* w = win + (size_t)p * M * M;
    {
        // batches of loads in flight before their LDS stores
        constexpr int NLD = (M * M + NT - 1) / NT, BATCH = NLD < 16 ? NLD : 16;
        static_assert(NLD % BATCH == 0, "load batches must divide the window");
#pragma unroll 1
        for (int k0 = 0; k0 < NLD; k0 += BATCH) {
            float2 ld[BATCH];
#pragma unroll
            for (int k = 0; k < BATCH; ++k) {
                const int idx = tid + (k0 + k) * NT;
                if (idx < M * M) ld[k] = w[idx];
            }
#pragma unroll
            for (int k = 0; k < BATCH; ++k) {
                const int idx = tid + (k0 + k) * NT;
                if (idx < M * M) buf[(idx / M) * RS + idx % M] = ld[k];
            }
        }
    }
    __syncthreads();
    typename F::Twiddles tw;
    tw.load(tw_m, lt);
    // rows, each exchanged in its own padded row
    for (int r0 = wave * G; r0 < M; r0 += NW * G) {
        float2* row = buf + (r0 + g) * RS;
        float2 v[E];
#pragma unroll
        for (int i = 0; i < E; ++i) v[i] = row[lt + LPT * i];
        F::template run_x<-1>(v, typename F::RowX{row}, tw, lt);
        F::sync();
#pragma unroll
        for (int i = 0; i < E; ++i) row[lt + LPT * i] = v[i];
    }
    __syncthreads();
    // columns, each exchanged in its own padded column, then intensity in place
    const float scale = 1.0f / ((float)M * (float)M * (float)M * (float)M);
    for (int c0 = wave * G; c0 < M; c0 += NW * G) {
        float2* col = buf + c0 + g;
        float2 v[E];
#pragma unroll
        for (int i = 0; i < E; ++i) v[i] = col[(lt + LPT * i) * RS];
        F::template run_x<-1>(v, typename F::template StrideX<RS>{col}, tw, lt);
        F::sync();
#pragma unroll
        for (int i = 0; i < E; ++i) col[(lt + LPT * i) * RS] = make_float2(cnorm(v[i]) * scale, 0.f);
    }
    __syncthreads();
    if (diff) {
        // the 4D output takes the same scale and accumulation as the 3D one
        float* d = diff + (size_t)p * M * M;
        for (int idx = tid; idx < M * M; idx += NT) {
            const float v = job.scale * buf[(idx / M) * RS + idx % M].x;
            d[idx] = job.accumulate ? d[idx] + v : v;
        }
    }
    if (!out) return;
    for (int b = wave; b < n_bins; b += NW) {
        float s = 0.f;
        for (int k = bin_start[b] + lane; k < bin_start[b + 1]; k += 64) {
            int pix = perm[k];
            s += buf[(pix / M) * RS + pix % M].x;
        }
        s = wave_sum(s);
        if (lane == 0) {
            float* o = out + (size_t)p * n_bins + b;
            *o = job.accumulate ? *o + job.scale * s : job.scale * s;
        }
    }
}

template <int M>
static hipError_t window_m(const WindowArgs* jobs, int n_jobs, hipStream_t st) {
    for (int j0 = 0; j0 < n_jobs; j0 += MAX_JOBS) {
        WindowBatch b{};
        b.n_jobs = n_jobs - j0 < MAX_JOBS ? n_jobs - j0 : MAX_JOBS;
        int blocks = 0;
        for (int k = 0; k < b.n_jobs; ++k) {
            const WindowArgs& a = jobs[j0 + k];
            b.job[k] = WindowJob{a.win, a.out, a.diff, a.perm, a.bin_start, a.tw_m, a.n_bins, blocks, a.scale,
                                 a.accumulate};
            blocks += a.n_probes;
        }
        if (blocks == 0) continue;
        hipLaunchKernelGGL((k_window_detect<M>), dim3((unsigned)blocks), dim3(WinCfg<M>::NT), 0, st, b);
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
__global__ __launch_bounds__(WG) void k_bin_reduce(const float* __restrict__ inten, int64_t pix_per_item,
                                                   float* __restrict__ out, const int* __restrict__ perm,
                                                   const int* __restrict__ bin_start, int n_bins, float scale,
                                                   int accumulate) {
    const int item = blockIdx.x;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const float* I = inten + (size_t)item * pix_per_item;
    for (int b = wave; b < n_bins; b += 4) {
        float s = 0.f;
        for (int k = bin_start[b] + lane; k < bin_start[b + 1]; k += 64) s += I[perm[k]];
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
    hipLaunchKernelGGL(k_bin_reduce, dim3((unsigned)n_items), dim3(WG), 0, st, inten, pix_per_item, out, perm,
                       bin_start, n_bins, scale, accumulate);
    return hipGetLastError();
}

}  // namespace prism
