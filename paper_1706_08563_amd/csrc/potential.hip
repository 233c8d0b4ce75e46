// potential.hip -- projected potential slices ("Calculation of the Projected
// Potentials", Fig. 1a-b).  Each atom adds its species' Gaussian terms
// A/(2 pi w^2) exp(-d^2/(2 w^2)) at minimum-image distance d < rc to the slab
// that holds it.
//
// One wavefront per (16 x 16 pixel tile, slice), 4 rows of one column per
// lane.  The atoms come sorted by (slice, cell of an nc x nc grid); the
// wavefront filters those of the cells within reach against the tile's
// bounding box (ballot compaction, so the list keeps the sorted order and the
// sums are deterministic).  A Gaussian is a product of one factor per axis,
// so a batch of listed atoms first fills a table of factors, 16 columns and 16
// rows per atom, and a pixel's term is one product of two table entries.
//
// Bound: VALU and LDS (a table read and 6 operations per pixel and atom).
// 51,000 atoms, 50 slices at 1024^2: 1.13 -> 0.38 ms against the form that
// tested every atom of the slice per tile and took two exponentials per pixel
// and atom (the 210 MB of V alone are 0.04 ms).  Tables of 8 atoms take 4.8 KB of
// LDS with two Gaussians, 33 wavefronts (8 per SIMD) of a CU's 160 KB; 16 atoms
// take the same time, 32 atoms 0.5 ms.
#include "kernels.hpp"

namespace prism {

constexpr int PT = 16;            // tile side (pixels)
constexpr int BATCH = 8;          // atoms per factor table
constexpr int PR = PT * PT / 64;  // pixels (rows) per lane

struct ListAtom { double dx, dy; int species; };   // offset from the tile centre

// NG: most Gaussians of a species.
template <int NG>
__global__ __launch_bounds__(64) void k_potential(float* __restrict__ V, int n, double L, int nc,
                                                  const PotAtom* __restrict__ atoms,
                                                  const int* __restrict__ cell_start,
                                                  const PotSpecies* __restrict__ species, float rc_max) {
    // an atom's factors along x (amplitudes included) and y, and squared distances
    __shared__ float f[2][BATCH][NG][PT], q[2][BATCH][PT];
    __shared__ float rc2[BATCH];
    __shared__ ListAtom list[BATCH + 64];
    const int ntx = n / PT, tile = blockIdx.x, s = blockIdx.y, lane = threadIdx.x;
    const double dx = L / n, inv_L = 1.0 / L;
    const double half = 0.5 * (PT - 1) * dx;
    const double cx = ((tile % ntx) * PT) * dx + half;      // tile centre
    const double cy = ((tile / ntx) * PT) * dx + half;
    const double lim = (double)rc_max + half * 1.0000001 + 1e-9;
    const int ix = lane % PT, iy0 = lane / PT;              // rows iy0 + 4 r
    float acc[PR];
#pragma unroll
    for (int r = 0; r < PR; ++r) acc[r] = 0.f;

    auto add_batch = [&](int first, int count) {
        __syncthreads();
        // factors of (atom k, position i of either axis)
        for (int t = lane; t < count * 2 * PT; t += 64) {
            const int k = t / (2 * PT), axis = (t / PT) % 2, i = t % PT;
            const ListAtom a = list[first + k];
            const PotSpecies& sp = species[a.species];
            // the distance in FP64: its rounding would be that of the offset
            double dd = i * dx - half - (axis ? a.dy : a.dx);
            dd -= L * rint(dd * inv_L);
            const float d = (float)dd, d2 = d * d;
            q[axis][k][i] = d2;
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const float e = expf(-d2 * sp.inv2w2[g]);
                f[axis][k][g][i] = axis ? e : (g < sp.n_gauss ? sp.amp_n[g] * e : 0.f);
            }
            if (t % (2 * PT) == 0) rc2[k] = sp.rc2;
        }
        __syncthreads();
        for (int k = 0; k < count; ++k) {
            const float lim2 = rc2[k] - q[0][k][ix];
            float ax[NG];
#pragma unroll
            for (int g = 0; g < NG; ++g) ax[g] = f[0][k][g][ix];
#pragma unroll
            for (int r = 0; r < PR; ++r) {
                const int iy = iy0 + r * (64 / PT);
                float v = 0.f;
#pragma unroll
                for (int g = 0; g < NG; ++g) v += ax[g] * f[1][k][g][iy];
                acc[r] += q[1][k][iy] < lim2 ? v : 0.f;
            }
        }
        __syncthreads();
    };

    // cells within reach of the tile, each once
    const double to_cell = nc * inv_L, reach = lim + 1e-9 * L;
    const int x0 = (int)floor((cx - reach) * to_cell), y0 = (int)floor((cy - reach) * to_cell);
    const int nx = min(nc, (int)floor((cx + reach) * to_cell) - x0 + 1);
    const int ny = min(nc, (int)floor((cy + reach) * to_cell) - y0 + 1);
    const int xa = ((x0 % nc) + nc) % nc;
    // lane j < ny: row j's cells xa .. xa + nx - 1, in up to two runs
    const int* row = cell_start + ((size_t)s * nc + ((y0 + lane) % nc + nc) % nc) * nc;
    int from[2] = {0, 0}, count[2] = {0, 0};
    if (lane < ny) {
        from[0] = row[xa];
        count[0] = row[min(xa + nx, nc)] - from[0];
        if (xa + nx > nc) {
            from[1] = row[0];
            count[1] = row[xa + nx - nc] - from[1];
        }
    }
    int total = count[0] + count[1];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) total += __shfl_xor(total, off, 64);
    int n_list = 0;
    for (int base = 0; base < total; base += 64) {
        // candidate base + lane of all runs
        int a = -1, before = base + lane;
        for (int j = 0; j < ny; ++j)
#pragma unroll
            for (int part = 0; part < 2; ++part) {
                const int c = __builtin_amdgcn_readlane(count[part], j);
                if (before >= 0 && before < c) a = __builtin_amdgcn_readlane(from[part], j) + before;
                before -= c;
            }
        bool near = false;
        ListAtom la{0.0, 0.0, 0};
        if (a >= 0) {
            const PotAtom at = atoms[a];
            double ddx = at.x - cx, ddy = at.y - cy;
            ddx -= L * rint(ddx * inv_L);
            ddy -= L * rint(ddy * inv_L);
            const double ex = fmax(fabs(ddx) - half, 0.0), ey = fmax(fabs(ddy) - half, 0.0);
            near = fabs(ddx) < lim && fabs(ddy) < lim && ex * ex + ey * ey < (double)rc_max * rc_max;
            la = ListAtom{ddx, ddy, at.species};
        }
        const unsigned long long mask = __ballot(near);
        if (near) list[n_list + __popcll(mask & ((1ull << lane) - 1ull))] = la;
        n_list += __popcll(mask);
        // the list holds under BATCH atoms before each addition of up to 64
        int done = 0;
        while (n_list - done >= BATCH) {
            add_batch(done, BATCH);
            done += BATCH;
        }
        if (done) {
            const int left = n_list - done;
            ListAtom keep{0.0, 0.0, 0};
            if (lane < left) keep = list[done + lane];
            __syncthreads();
            if (lane < left) list[lane] = keep;
            n_list = left;
        }
    }
    if (n_list) add_batch(0, n_list);
    const int px = (tile % ntx) * PT + ix, py = (tile / ntx) * PT + iy0;
#pragma unroll
    for (int r = 0; r < PR; ++r) V[((size_t)s * n + py + r * (64 / PT)) * n + px] = acc[r];
}

hipError_t launch_potential(float* V, int n, int n_slices, double L, int cells, const PotAtom* atoms,
                            const int* cell_start, const PotSpecies* species, int max_gauss, float rc_max,
                            hipStream_t st) {
    dim3 grid((unsigned)((n / PT) * (n / PT)), (unsigned)n_slices);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(64), 0, st, V, n, L, cells, atoms, cell_start, species, rc_max);
    };
    if (max_gauss <= 2) launch(k_potential<2>);
    else launch(k_potential<4>);
    return hipGetLastError();
}

}  // namespace prism
