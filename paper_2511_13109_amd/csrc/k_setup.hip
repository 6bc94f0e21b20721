// Hierarchy setup: viscosity-variation flags, compaction of the flagged
// elements, local Galerkin blocks (paper eqs. (2.6)-(2.7), (B.2)) and the
// Jacobi diagonals of the level operators (eq. (2.9)).
#include <hip/hip_runtime.h>
#include <hipcub/hipcub.hpp>

#include "gca_math.h"
#include "internal.h"

namespace agca {
namespace {

constexpr int NT = 256;

inline unsigned grid_for(int64_t n) { return (unsigned)((n + NT - 1) / NT); }

// Macro-element granularity (eqs. (2.8)-(2.9)).  A level-l element (cell c, order s)
// lies in the macro cube c >> l; inside that cube the Kuhn simplex with axis order
// (a1, a2, a3) is the set x_a1 >= x_a2 >= x_a3 of relative coordinates, so the macro
// simplex holding the element is the descending order of its centroid's relative
// coordinates.  In units of a quarter level-l cell that centroid is 4 (c - corner)
// plus 3, 2, 1 along the element's own a1, a2, a3: integers with distinct residues
// mod 4, hence never tied.
__device__ __forceinline__ int macro_of(int64_t e, int n, int l) {
    const int s = (int)(e % 6);
    int64_t c = e / 6;
    const int cx = (int)(c % n), cy = (int)((c / n) % n), cz = (int)(c / ((int64_t)n * n));
    const int mx = cx >> l, my = cy >> l, mz = cz >> l;
    auto w = [&](int ax) { return ax == axis1(s) ? 3 : (ax == axis2(s) ? 2 : 1); };
    const int r0 = 4 * (cx - (mx << l)) + w(0);
    const int r1 = 4 * (cy - (my << l)) + w(1);
    const int r2 = 4 * (cz - (mz << l)) + w(2);
    const int a1 = (r0 > r1) ? (r0 > r2 ? 0 : 2) : (r1 > r2 ? 1 : 2);
    const int a3 = (r0 < r1) ? (r0 < r2 ? 0 : 2) : (r1 < r2 ? 1 : 2);
    return order_index(a1, 3 - a1 - a3, a3) + 6 * (mx + 2 * (my + 2 * mz));
}

// Flags and effective coefficients.  For every element of a coarse level the minimum,
// maximum and mean of the finest coefficient over its finest descendants, built bottom-up:
// min and max are exact, so the pyramid equals the direct definition of the strict ratio test
// in FP64; all descendants have the same volume, so the mean of the children's means is the
// mean.  A flagged element's operator is its DCA matrix with that mean: for P1 functions the
// Galerkin product (eq. (2.7)) sums the finest element matrices nu_d K_d of its descendants
// against the constant gradients of the coarse hat functions.  Bound by the reads of the
// level below (8 children in runs of up to 48 bytes).  FROM_FINE: the three inputs are the
// finest coefficient.
template <bool FROM_FINE>
__global__ void __launch_bounds__(NT)
k_coarsen(int n, int l, const double* __restrict__ mn_f, const double* __restrict__ mx_f,
          const double* __restrict__ mean_f, int mode, double tau, uint64_t bits, double* __restrict__ mn,
          double* __restrict__ mx, double* __restrict__ mean, int32_t* __restrict__ flag, double* __restrict__ nu) {
    const int64_t ne = 6LL * n * n * n;
    const int64_t e = blockIdx.x * (int64_t)NT + threadIdx.x;
    if (e >= ne) return;
    const int64_t cells_f = 8LL * n * n * n;
    double a = INFINITY, b = -INFINITY, s = 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int64_t id = child_id(n, e, k), c = FROM_FINE ? elem_index(id, cells_f) : id;
        const double v = mn_f[c];
        a = fmin(a, v);
        b = fmax(b, FROM_FINE ? v : mx_f[c]);
        s += FROM_FINE ? v : mean_f[c];
    }
    s *= 0.125;
    mn[e] = a;
    mx[e] = b;
    mean[e] = s;
    const bool f = mode == AGCA_FLAG_ALL || (mode == AGCA_FLAG_RATIO && b > tau * a) ||
                   (mode == AGCA_FLAG_MACRO && ((bits >> macro_of(e, n, l)) & 1u));
    flag[e] = f ? 1 : 0;
    if (f) nu[elem_index(e, ne / 6)] = s;
}

// max over the finest elements of each macro element of |grad eta_h| (P1 interpolant):
// along the path of simplex s the gradient components are n (eta(k_j) - eta(k_{j-1}))
// on axis a_j.  Norms are >= 0, so the maximum of their bit patterns as unsigned
// integers is the maximum of the values (exact and order-independent).
__global__ void __launch_bounds__(NT)
k_macro_grad_max(int n, int l, const double* __restrict__ eta, unsigned long long* __restrict__ gbits) {
    __shared__ unsigned long long loc[48];
    if (threadIdx.x < 48) loc[threadIdx.x] = 0ull;
    __syncthreads();
    const int64_t ne = 6LL * n * n * n;
    const int64_t n1 = n + 1;
    const double scale = (double)n;
    for (int64_t e = blockIdx.x * (int64_t)NT + threadIdx.x; e < ne; e += (int64_t)gridDim.x * NT) {
        const int s = (int)(e % 6);
        const int64_t c = e / 6;
        const int64_t cx = c % n, cy = (c / n) % n, cz = c / ((int64_t)n * n);
        const int64_t base = cx + n1 * (cy + n1 * cz);
        double v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = path_corner(s, j);
            v[j] = eta[base + (k & 1) + n1 * (((k >> 1) & 1) + n1 * (k >> 2))];
        }
        const double g1 = scale * (v[1] - v[0]), g2 = scale * (v[2] - v[1]), g3 = scale * (v[3] - v[2]);
        const double nrm = sqrt(g1 * g1 + g2 * g2 + g3 * g3);
        atomicMax(&loc[macro_of(e, n, l)], (unsigned long long)__double_as_longlong(nrm));
    }
    __syncthreads();
    if (threadIdx.x < 48 && loc[threadIdx.x] != 0ull) atomicMax(&gbits[threadIdx.x], loc[threadIdx.x]);
}

__global__ void __launch_bounds__(NT)
k_scatter_ids(int64_t ne, const int32_t* __restrict__ flag, const int32_t* __restrict__ pos,
              int32_t* __restrict__ blk, int32_t* __restrict__ ids, int64_t* __restrict__ count) {
    const int64_t e = blockIdx.x * (int64_t)NT + threadIdx.x;
    if (e >= ne) return;
    const int32_t f = flag[e];
    const int32_t p = pos[e];
    blk[e] = f ? p : -1;
    if (f) ids[p] = (int32_t)e;
    if (e == ne - 1) *count = (int64_t)p + f;
}

// ---------------------------------------------------------------------------
// Local Galerkin blocks.  Component block (c,d) of an element's block follows
// the scalar recursion (B.2):  G_m = sum_k P_k^T G_child(k) P_k, with the
// constant local interpolations P_k of kuhn.h, down to the finest level where
// G is the element matrix nu_e (h/6) K(s).  One thread per (element, c, d).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void store_block(double* __restrict__ dst, int M, int c, int d,
                                            const double (&G)[16]) {
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) dst[(4 * c + a) * M + 4 * d + b] = G[4 * a + b];
}

__global__ void __launch_bounds__(NT)
k_gca_fused2(int ncomp, int n, const double* __restrict__ nu_fine, double w_scale,
             const int32_t* __restrict__ blk_child, double* __restrict__ blocks_child,
             const int32_t* __restrict__ blk_self, double* __restrict__ blocks_self,
             double* __restrict__ trans_out) {
    const int64_t ne = 6LL * n * n * n;
    const int ncc = ncomp * ncomp;
    const int64_t t = blockIdx.x * (int64_t)NT + threadIdx.x;
    if (t >= ne * ncc) return;
    const int64_t e = t / ncc;
    const int cd = (int)(t % ncc);
    const int c = cd / ncomp, d = cd % ncomp;
    const int M = 4 * ncomp;
    const int64_t cells_f = 64LL * n * n * n;
    double Ge[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) Ge[i] = 0.0;
    for (int k = 0; k < 8; ++k) {
        const int64_t ce = child_id(n, e, k);
        double Gc[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) Gc[i] = 0.0;
        for (int kk = 0; kk < 8; ++kk) {
            const int64_t ge = child_id(2 * n, ce, kk);
            double K[16];
            fine_block(ncomp, (int)(ge % 6), c, d, nu_fine[elem_index(ge, cells_f)] * w_scale, K);
            add_ptkp(kk, K, Gc);
        }
        const int32_t bc = blk_child[ce];
        if (bc >= 0) store_block(blocks_child + (int64_t)bc * M * M, M, c, d, Gc);
        add_ptkp(k, Gc, Ge);
    }
    const int32_t bs = blk_self[e];
    if (bs >= 0) store_block(blocks_self + (int64_t)bs * M * M, M, c, d, Ge);
    if (trans_out) store_block(trans_out + e * M * M, M, c, d, Ge);
}

__global__ void __launch_bounds__(NT)
k_gca_from_fine(int ncomp, int n, int64_t nflag, const int32_t* __restrict__ ids,
                const double* __restrict__ nu_fine, double w_scale, double* __restrict__ blocks) {
    const int ncc = ncomp * ncomp;
    const int64_t t = blockIdx.x * (int64_t)NT + threadIdx.x;
    if (t >= nflag * ncc) return;
    const int64_t i = t / ncc;
    const int cd = (int)(t % ncc);
    const int c = cd / ncomp, d = cd % ncomp;
    const int M = 4 * ncomp;
    const int64_t e = ids[i];
    const int64_t cells_f = 8LL * n * n * n;
    double G[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) G[q] = 0.0;
    for (int k = 0; k < 8; ++k) {
        const int64_t ge = child_id(n, e, k);
        double K[16];
        fine_block(ncomp, (int)(ge % 6), c, d, nu_fine[elem_index(ge, cells_f)] * w_scale, K);
        add_ptkp(k, K, G);
    }
    store_block(blocks + i * M * M, M, c, d, G);
}

__global__ void __launch_bounds__(NT)
k_gca_up(int ncomp, int n, const double* __restrict__ trans_in, const int32_t* __restrict__ blk_self,
         double* __restrict__ blocks_self, double* __restrict__ trans_out) {
    const int64_t ne = 6LL * n * n * n;
    const int ncc = ncomp * ncomp;
    const int64_t t = blockIdx.x * (int64_t)NT + threadIdx.x;
    if (t >= ne * ncc) return;
    const int64_t e = t / ncc;
    const int cd = (int)(t % ncc);
    const int c = cd / ncomp, d = cd % ncomp;
    const int M = 4 * ncomp;
    double G[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) G[q] = 0.0;
    for (int k = 0; k < 8; ++k) {
        const int64_t ce = child_id(n, e, k);
        const double* src = trans_in + ce * M * M;
        double K[16];
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) K[4 * a + b] = src[(4 * c + a) * M + 4 * d + b];
        add_ptkp(k, K, G);
    }
    const int32_t bs = blk_self[e];
    if (bs >= 0) store_block(blocks_self + (int64_t)bs * M * M, M, c, d, G);
    if (trans_out) store_block(trans_out + e * M * M, M, c, d, G);
}

// ---------------------------------------------------------------------------
// Diagonal of a level operator: each node gathers the diagonal entries of the
// (up to 24) simplices that contain it.  Boundary nodes get 0.
// ---------------------------------------------------------------------------
template <int NC>
__global__ void __launch_bounds__(NT)
k_diagonal(int n, const double* __restrict__ nu, double scale, double* __restrict__ diag) {
    const int64_t n1 = n + 1, N = n1 * n1 * n1;
    const int64_t p = blockIdx.x * (int64_t)NT + threadIdx.x;
    if (p >= N) return;
    const int x = (int)(p % n1), y = (int)((p / n1) % n1), z = (int)(p / (n1 * n1));
    const bool bd = x == 0 || y == 0 || z == 0 || x == n || y == n || z == n;
    const int64_t cells = (int64_t)n * n * n;
    double acc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = 0.0;
    if (!bd) {
        for (int k = 0; k < 8; ++k) {
            const int cx = x - (k & 1), cy = y - ((k >> 1) & 1), cz = z - ((k >> 2) & 1);
            const int64_t cell = cx + (int64_t)n * (cy + (int64_t)n * cz);
            for (int s = 0; s < 6; ++s) {
                int a = -1;
                for (int j = 0; j < 4; ++j)
                    if (path_corner(s, j) == k) a = j;
                if (a < 0) continue;
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    acc[c] += nu[elem_slot(s, cell, cells)] * scale * (double)elem_entry(NC, s, c, a, c, a);
            }
        }
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) diag[c * N + p] = acc[c];
}

template <typename T>
__global__ void __launch_bounds__(NT)
k_invert_diag(int64_t count, const double* __restrict__ diag, T* __restrict__ dinv) {
    const int64_t i = blockIdx.x * (int64_t)NT + threadIdx.x;
    if (i >= count) return;
    const double d = diag[i];
    dinv[i] = d > 0.0 ? T(1.0 / d) : T(0);
}

}  // namespace

hipError_t launch_coarsen(int n, int l, const double* mn_f, const double* mx_f, const double* mean_f, int mode,
                          double tau, uint64_t bits, double* mn, double* mx, double* mean, int32_t* flag,
                          double* nu, hipStream_t st) {
    if (!mn_f || !mx_f || !mean_f || !mn || !mx || !mean || !flag || !nu || n != (2 << l)) return hipErrorInvalidValue;
    const int64_t ne = 6LL * n * n * n;
    if (mn_f == mx_f)
        hipLaunchKernelGGL(k_coarsen<true>, dim3(grid_for(ne)), dim3(NT), 0, st, n, l, mn_f, mx_f, mean_f, mode, tau,
                           bits, mn, mx, mean, flag, nu);
    else
        hipLaunchKernelGGL(k_coarsen<false>, dim3(grid_for(ne)), dim3(NT), 0, st, n, l, mn_f, mx_f, mean_f, mode, tau,
                           bits, mn, mx, mean, flag, nu);
    return hipGetLastError();
}
hipError_t launch_macro_grad_max(int L, const double* eta, unsigned long long* gbits, hipStream_t st) {
    if (!eta || !gbits || L < 0 || L > 12) return hipErrorInvalidValue;
    const int n = 2 << L;
    const int64_t ne = 6LL * n * n * n;
    const unsigned blocks = (unsigned)std::min<int64_t>((ne + NT - 1) / NT, 4096);
    hipLaunchKernelGGL(k_macro_grad_max, dim3(blocks), dim3(NT), 0, st, n, L, eta, gbits);
    return hipGetLastError();
}
hipError_t compact_scratch_bytes(int64_t ne, size_t* bytes) {
    size_t tmp = 0;
    hipError_t err = hipcub::DeviceScan::ExclusiveSum(nullptr, tmp, (const int32_t*)nullptr,
                                                      (int32_t*)nullptr, (int)ne);
    *bytes = tmp + (size_t)ne * sizeof(int32_t) + 256;
    return err;
}
hipError_t launch_compact(int64_t ne, const int32_t* flag, int32_t* blk, int32_t* ids, int64_t* count_dev, void* scratch, size_t scratch_bytes,
                          hipStream_t st) {
    if (!flag || !blk || !ids || !count_dev || !scratch) return hipErrorInvalidValue;
    // scratch: [pos (ne int32, 256-aligned)] [cub temp]
    int32_t* pos = static_cast<int32_t*>(scratch);
    size_t off = (((size_t)ne * sizeof(int32_t)) + 255) & ~(size_t)255;
    void* tmp = static_cast<char*>(scratch) + off;
    size_t tmp_bytes = scratch_bytes - off;
    hipError_t err = hipcub::DeviceScan::ExclusiveSum(tmp, tmp_bytes, flag, pos, (int)ne, st);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(k_scatter_ids, dim3(grid_for(ne)), dim3(NT), 0, st, ne, flag, pos, blk, ids, count_dev);
    return hipGetLastError();
}
hipError_t launch_gca_fused2(int ncomp, int n, const double* nu_fine, double h_fine,
                             const int32_t* blk_child, double* blocks_child,
                             const int32_t* blk_self, double* blocks_self, double* trans_out,
                             hipStream_t st) {
    if (!nu_fine || !blk_child || !blk_self) return hipErrorInvalidValue;
    const int64_t threads = 6LL * n * n * n * ncomp * ncomp;
    hipLaunchKernelGGL(k_gca_fused2, dim3(grid_for(threads)), dim3(NT), 0, st, ncomp, n, nu_fine,
                       h_fine / 6.0, blk_child, blocks_child, blk_self, blocks_self, trans_out);
    return hipGetLastError();
}
hipError_t launch_gca_from_fine(int ncomp, int n, int64_t nflag, const int32_t* ids,
                                const double* nu_fine, double h_fine, double* blocks,
                                hipStream_t st) {
    const int64_t threads = nflag * ncomp * ncomp;
    if (threads == 0) return hipSuccess;
    hipLaunchKernelGGL(k_gca_from_fine, dim3(grid_for(threads)), dim3(NT), 0, st, ncomp, n, nflag,
                       ids, nu_fine, h_fine / 6.0, blocks);
    return hipGetLastError();
}
hipError_t launch_gca_up(int ncomp, int n, const double* trans_in, const int32_t* blk_self,
                         double* blocks_self, double* trans_out, hipStream_t st) {
    if (!trans_in || !blk_self) return hipErrorInvalidValue;
    const int64_t threads = 6LL * n * n * n * ncomp * ncomp;
    hipLaunchKernelGGL(k_gca_up, dim3(grid_for(threads)), dim3(NT), 0, st, ncomp, n, trans_in,
                       blk_self, blocks_self, trans_out);
    return hipGetLastError();
}
hipError_t launch_diagonal(int ncomp, int n, const double* nu, double scale, double* diag, hipStream_t st) {
    if (!nu || !diag) return hipErrorInvalidValue;
    const int64_t N = (int64_t)(n + 1) * (n + 1) * (n + 1);
    if (ncomp == 1)
        hipLaunchKernelGGL(k_diagonal<1>, dim3(grid_for(N)), dim3(NT), 0, st, n, nu, scale, diag);
    else
        hipLaunchKernelGGL(k_diagonal<3>, dim3(grid_for(N)), dim3(NT), 0, st, n, nu, scale, diag);
    return hipGetLastError();
}
template <typename T>
hipError_t launch_invert_diag(int64_t count, const double* diag, T* dinv, hipStream_t st) {
    if (!diag || !dinv) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_invert_diag<T>, dim3(grid_for(count)), dim3(NT), 0, st, count, diag, dinv);
    return hipGetLastError();
}
template hipError_t launch_invert_diag<double>(int64_t, const double*, double*, hipStream_t);
template hipError_t launch_invert_diag<float>(int64_t, const double*, float*, hipStream_t);

}  // namespace agca
