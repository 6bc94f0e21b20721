// Geometric multigrid for the BFBT pressure operator Z = B W^-1 B^T (eq. (4.2)) on the
// pressure lattice: stencil products, damped Jacobi, probing assembly of the stencils
// and the 27-node coarse solve.  Stencil layout and the probing colours: zstencil.h.
//
// The stencil kernels are bound by memory: a node reads its 33 stored stencil entries (264
// bytes; the 32 lower entries are its neighbours' stored ones, read again from cache) and
// writes one value.  One thread per node, consecutive threads along x.
#include <hip/hip_runtime.h>

#include "internal.h"
#include "kuhn.h"
#include "zstencil.h"

namespace agca {
namespace {

constexpr int NT = 256;
constexpr int kZThreads = 576;  // largest workgroup of the stencil kernel (9 wavefronts)

unsigned grid_for(int64_t n) { return (unsigned)((n + NT - 1) / NT); }

// MODE 0: out = S x;  1: out = r - S x;  2 (damped Jacobi): out = x + omega (r - S x) / S_c.
// S: the stored half of a symmetric stencil over the padded lattice (zstencil.h).  Each
// stored offset o contributes twice: S_o(k) x(k + o) and, for the lower offset -o,
// S_o(k - o) x(k - o), the second entry being the neighbour's own.  x counts 0 outside the
// lattice, where the stencil entries are 0 as well (written by the assembly, or padding).
//
// A workgroup owns `rows` whole rows of nodes of one plane, one node per thread, with x on
// the five planes around them in LDS.  The kernel is bound by two things at once (129^3
// nodes, counters of the form that read x through the cache and dealt the workgroups to the
// XCDs in turn): the address unit of the vector memory path, 130 loads per node, busy 83 %
// of the time; and the memory behind L2, 1.27 GB per pass against the stencil's 0.62 GB,
// because most neighbours' entries were read by another XCD.  x in LDS halves the loads; and
// every XCD owns a slab of planes and takes it row group by row group, all planes of a group
// before the next group, so that the workgroups that share an entry run at the same time on
// the same XCD (0.79 GB).  Pass at 129^3 nodes 196 -> 165 us, one V-cycle 1093 -> 940 us, the
// BFBT application at 257^3 velocity nodes 12.4 -> 10.9 ms.  Interleaving a row's 33 entries
// (one stream instead of 33) made no difference.
template <int MODE>
__global__ void __launch_bounds__(kZThreads)
k_zstencil(int n, int rows, int gy, const double* __restrict__ S, const double* __restrict__ x,
           const double* __restrict__ r, double omega, double* __restrict__ out) {
    extern __shared__ double xl[];  // [5 planes][rows + 4][n + 5]
    const int n1 = n + 1, np1 = n + 1 + 2 * kZPad;
    const size_t NP = (size_t)np1 * np1 * np1;
    // XCD b % 8 owns the planes [z0, z1); its workgroups: group slowest, plane fastest
    const int xcd = blockIdx.x & 7, q = blockIdx.x >> 3;
    const int z0 = xcd * n1 / 8, z1 = (xcd + 1) * n1 / 8, planes = (n1 + 7) / 8;
    const int group = q / planes, z = z0 + (q - group * planes);
    if (z >= z1) return;
    const int Y0 = group * rows;
    const int lw = n1 + 4, lp = lw * (rows + 4);
    const int tid = threadIdx.x, nt = blockDim.x;
    const int ty = tid / n1, tx = tid - ty * n1;
    // x around the tile: every thread its own node of the five planes and at most a few of
    // the frame's (two rows and columns on every side), all loads of a position in flight
    auto stage = [&](int dx, int dy) {
        const int px = dx - 2, py = Y0 + dy - 2;
        const bool in = (unsigned)px <= (unsigned)n && (unsigned)py <= (unsigned)n;
        const double* xr = x + (in ? px + (int64_t)n1 * py : 0);
        double v[5];
#pragma unroll
        for (int d = 0; d < 5; ++d) {
            const int pz = z + d - 2;
            v[d] = xr[(int64_t)min(max(pz, 0), n) * n1 * n1];
            if (!in || pz < 0 || pz > n) v[d] = 0.0;
        }
#pragma unroll
        for (int d = 0; d < 5; ++d) xl[d * lp + dy * lw + dx] = v[d];
    };
    if (ty < rows) stage(tx + 2, ty + 2);
    const int frame = 4 * lw + 4 * rows;
    for (int i = tid; i < frame; i += nt) {
        if (i < 4 * lw) {
            const int row = i / lw;
            stage(i - row * lw, row < 2 ? row : rows + row);
        } else {
            const int k = i - 4 * lw, col = k & 3;
            stage(col < 2 ? col : n1 + col, 2 + (k >> 2));
        }
    }
    __syncthreads();
    const int py = Y0 + ty;
    if (ty >= rows || py > n) return;
    const uint32_t p = (uint32_t)tx + (uint32_t)n1 * ((uint32_t)py + (uint32_t)n1 * (uint32_t)z);
    const uint32_t kp = (uint32_t)(tx + kZPad) +
                        (uint32_t)np1 * ((uint32_t)(py + kZPad) + (uint32_t)np1 * (uint32_t)(z + kZPad));
    const double* xc = xl + 2 * lp + (ty + 2) * lw + tx + 2;
    const double sc = S[kp];
    double acc = sc * xc[0];
#pragma unroll
    for (int j = 1; j < kZStored; ++j) {
        const int i = kZCentre + j;
        const int dx = kZTable.dx[i], dy = kZTable.dy[i], dz = kZTable.dz[i];
        const int64_t dp = dx + (int64_t)np1 * (dy + (int64_t)np1 * dz);
        const double* Sj = S + (size_t)j * NP;
        const int o = dx + lw * dy + lp * dz;
        acc = fma(Sj[kp], xc[o], acc);
        acc = fma((Sj - dp)[kp], xc[-o], acc);
    }
    if (MODE == 0)
        out[p] = acc;
    else if (MODE == 1)
        out[p] = r[p] - acc;
    else
        out[p] = xc[0] + omega * (r[p] - acc) / sc;
}

// first Jacobi sweep from a zero guess: out = omega r / S_c
__global__ void __launch_bounds__(NT)
k_zjacobi0(int n, const double* __restrict__ S, const double* __restrict__ r, double omega,
           double* __restrict__ out) {
    const int n1 = n + 1, np1 = n + 1 + 2 * kZPad;
    const int64_t N = (int64_t)n1 * n1 * n1;
    const int64_t p = blockIdx.x * (int64_t)NT + threadIdx.x;
    if (p >= N) return;
    int px, py, pz;
    node_coords(p, n, px, py, pz);
    const int64_t kp = (px + kZPad) + (int64_t)np1 * ((py + kZPad) + (int64_t)np1 * (pz + kZPad));
    out[p] = omega * r[p] / S[kp];
}

// indicator of the nodes of probing colour c
__global__ void __launch_bounds__(NT)
k_zprobe(int n, int c, double* __restrict__ out) {
    const int64_t N = (int64_t)(n + 1) * (n + 1) * (n + 1);
    const int64_t p = blockIdx.x * (int64_t)NT + threadIdx.x;
    if (p >= N) return;
    int px, py, pz;
    node_coords(p, n, px, py, pz);
    out[p] = z_colour(px, py, pz) == c ? 1.0 : 0.0;
}

// y = Z (indicator of colour c): at node k it is Z(k, k + o) for the one offset o whose
// node k + o has colour c; stored when o is one of the stored offsets (0 where k + o
// leaves the lattice).  A lower offset's value is the stored entry of node k + o
// (symmetry), probed with the colour of k, so each stored entry is written once.
__global__ void __launch_bounds__(NT)
k_zextract(int n, int c, const double* __restrict__ y, double* __restrict__ S) {
    const int n1 = n + 1, np1 = n + 1 + 2 * kZPad;
    const int64_t N = (int64_t)n1 * n1 * n1;
    const size_t NP = (size_t)np1 * np1 * np1;
    const int64_t p = blockIdx.x * (int64_t)NT + threadIdx.x;
    if (p >= N) return;
    int px, py, pz;
    node_coords(p, n, px, py, pz);
    const int want = z_colour_mod(c - z_colour(px, py, pz));
    int oi = 0, dx = 0, dy = 0, dz = 0;
#pragma unroll
    for (int i = 0; i < kZOffsets; ++i)
        if (z_colour(kZTable.dx[i], kZTable.dy[i], kZTable.dz[i]) == want) {
            oi = i;
            dx = kZTable.dx[i];
            dy = kZTable.dy[i];
            dz = kZTable.dz[i];
        }
    if (oi < kZCentre) return;
    const bool in = (unsigned)(px + dx) <= (unsigned)n && (unsigned)(py + dy) <= (unsigned)n &&
                    (unsigned)(pz + dz) <= (unsigned)n;
    const int64_t kp = (px + kZPad) + (int64_t)np1 * ((py + kZPad) + (int64_t)np1 * (pz + kZPad));
    S[(size_t)(oi - kZCentre) * NP + kp] = in ? y[p] : 0.0;
}

// the full 65-offset form of a stored stencil: out[i N + k] = Z(k, k + o_i)
__global__ void __launch_bounds__(NT)
k_zexpand(int n, const double* __restrict__ S, double* __restrict__ out) {
    const int n1 = n + 1, np1 = n + 1 + 2 * kZPad;
    const int64_t N = (int64_t)n1 * n1 * n1;
    const size_t NP = (size_t)np1 * np1 * np1;
    const int64_t p = blockIdx.x * (int64_t)NT + threadIdx.x;
    if (p >= N) return;
    int px, py, pz;
    node_coords(p, n, px, py, pz);
    const int64_t kp = (px + kZPad) + (int64_t)np1 * ((py + kZPad) + (int64_t)np1 * (pz + kZPad));
#pragma unroll
    for (int i = 0; i < kZOffsets; ++i) {
        const int dx = kZTable.dx[i], dy = kZTable.dy[i], dz = kZTable.dz[i];
        const int64_t dp = dx + (int64_t)np1 * (dy + (int64_t)np1 * dz);
        // o_i stored (i >= 32) at node k; a lower o_i as -o_i = o_{64-i} at node k + o_i
        out[i * N + p] = i >= kZCentre ? S[(size_t)(i - kZCentre) * NP + kp]
                                       : S[(size_t)(kZOffsets - 1 - i - kZCentre) * NP + kp + dp];
    }
}

// y = M r on the 27 nodes of level 0 (M row-major 27 x 27)
__global__ void __launch_bounds__(64)
k_zcoarse(const double* __restrict__ M, const double* __restrict__ r, double* __restrict__ y) {
    const int t = threadIdx.x;
    if (t >= 27) return;
    double acc = 0.0;
    for (int j = 0; j < 27; ++j) acc = fma(M[t * 27 + j], r[j], acc);
    y[t] = acc;
}

}  // namespace

hipError_t launch_zstencil(int mode, int n, const double* S, const double* x, const double* r,
                           double omega, double* out, hipStream_t st) {
    if (n < 1 || !S || !x || !out || (mode != 0 && !r) || mode < 0 || mode > 2 || x == out)
        return hipErrorInvalidValue;
    if ((int64_t)(n + 1) * (n + 1) * (n + 1) > (int64_t)UINT32_MAX / 8) return hipErrorInvalidValue;
    // whole rows, as many per workgroup as leave the fewest idle lanes (129 nodes: 4 rows on 9
    // wavefronts) within 64 KB of LDS, which keeps at least two workgroups per compute unit
    const int n1 = n + 1;
    if (n1 > kZThreads) return hipErrorInvalidValue;
    auto lds_of = [&](int c) { return 5 * sizeof(double) * (size_t)(n1 + 4) * (size_t)(c + 4); };
    int rows = 1;
    double best = 0.0;
    for (int c = 1; c <= 32 && c <= n1 && c * n1 <= kZThreads && lds_of(c) <= 65536; ++c) {
        const double lanes = (double)(c * n1) / (64 * ((c * n1 + 63) / 64));
        if (lanes > best) {
            best = lanes;
            rows = c;
        }
    }
    const int gy = (n1 + rows - 1) / rows, threads = 64 * ((rows * n1 + 63) / 64);
    const unsigned g = 8u * (unsigned)gy * (unsigned)((n1 + 7) / 8);
    const size_t lds = lds_of(rows);
    if (lds > 65536) {
        const void* f = mode == 0 ? (const void*)k_zstencil<0> : mode == 1 ? (const void*)k_zstencil<1> : (const void*)k_zstencil<2>;
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
#define AGCA_Z(M) hipLaunchKernelGGL(k_zstencil<M>, dim3(g), dim3(threads), lds, st, n, rows, gy, S, x, r, omega, out)
    if (mode == 0)
        AGCA_Z(0);
    else if (mode == 1)
        AGCA_Z(1);
    else
        AGCA_Z(2);
#undef AGCA_Z
    return hipGetLastError();
}

hipError_t launch_zjacobi0(int n, const double* S, const double* r, double omega, double* out,
                           hipStream_t st) {
    if (n < 1 || !S || !r || !out) return hipErrorInvalidValue;
    const int64_t N = (int64_t)(n + 1) * (n + 1) * (n + 1);
    hipLaunchKernelGGL(k_zjacobi0, dim3(grid_for(N)), dim3(NT), 0, st, n, S, r, omega, out);
    return hipGetLastError();
}

hipError_t launch_zexpand(int n, const double* S, double* out, hipStream_t st) {
    if (n < 1 || !S || !out) return hipErrorInvalidValue;
    const int64_t N = (int64_t)(n + 1) * (n + 1) * (n + 1);
    hipLaunchKernelGGL(k_zexpand, dim3(grid_for(N)), dim3(NT), 0, st, n, S, out);
    return hipGetLastError();
}

hipError_t launch_zprobe(int n, int colour, double* out, hipStream_t st) {
    if (n < 1 || colour < 0 || colour >= kZColours || !out) return hipErrorInvalidValue;
    const int64_t N = (int64_t)(n + 1) * (n + 1) * (n + 1);
    hipLaunchKernelGGL(k_zprobe, dim3(grid_for(N)), dim3(NT), 0, st, n, colour, out);
    return hipGetLastError();
}

hipError_t launch_zextract(int n, int colour, const double* y, double* S, hipStream_t st) {
    if (n < 1 || colour < 0 || colour >= kZColours || !y || !S) return hipErrorInvalidValue;
    const int64_t N = (int64_t)(n + 1) * (n + 1) * (n + 1);
    hipLaunchKernelGGL(k_zextract, dim3(grid_for(N)), dim3(NT), 0, st, n, colour, y, S);
    return hipGetLastError();
}

hipError_t launch_zcoarse(const double* M, const double* r, double* y, hipStream_t st) {
    if (!M || !r || !y || r == y) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_zcoarse, dim3(1), dim3(64), 0, st, M, r, y);
    return hipGetLastError();
}

}  // namespace agca
