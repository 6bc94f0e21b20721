// Generalized Stokes pieces (paper Section 3.1, eqs. (3.3)-(3.5)): velocity P1 on the
// finest level L (P1-iso-P2), pressure P1 on level L-1 with every node of that level a
// degree of freedom.
//
//   B = - integral psi_k div Phi_j = -P^T B_L,
//   (B_L u)_v = sum over the simplices d containing v of |d|/4 div_d(u),
// because psi_k is linear on every fine simplex (its mean over d is the mean of its
// vertex values, which the interpolation P of eq. (2.4) gives).  On the Kuhn lattice
// |d| = h^3/6 and the barycentric gradients are grad(s, a, c) / h (kuhn.h), so
//   (B_L u)_v = h^2/24 sum_{d containing v} sum_{b, c} grad(s, b, c) u_c(b).
// B^T p = -B_L^T (P p).  The pressure preconditioner is the lumped mass weighted by
// 1/nu, m = P^T m_L, m_L(v) = h^3/24 sum_{d containing v} 1/nu_d.
//
// Every kernel gathers per node (no atomics): the simplices around a node are the
// ones of the 8 cells sharing it whose path passes through it, and their vertices
// are the node's 15 lattice neighbours (kuhn.h nbr_of).
#include <hip/hip_runtime.h>

#include "cube_tile.h"
#include "internal.h"
#include "kuhn.h"

namespace agca {
namespace {

constexpr int NT = 256;

__device__ __forceinline__ void node_xyz(int64_t p, int n, int& x, int& y, int& z) {
    node_coords(p, n, x, y, z);
}

// cell of node (x,y,z) that has the node as its corner k, and whether it exists
__device__ __forceinline__ bool cell_of(int n, int x, int y, int z, int k, int64_t& cell) {
    const int cx = x - (k & 1), cy = y - ((k >> 1) & 1), cz = z - ((k >> 2) & 1);
    cell = cx + (int64_t)n * (cy + (int64_t)n * cz);
    return cx >= 0 && cy >= 0 && cz >= 0 && cx < n && cy < n && cz < n;
}

// B_L and its transpose have constant coefficients: the sums over the simplices around a node
// collapse to one number per neighbour and component.  (B_L at a boundary node sums over fewer
// cells, but the cells that are missing have no interior vertex, and the velocity is 0 elsewhere.)
constexpr int nbr_index(int dx, int dy, int dz) {  // kuhn.h neighbour index of an offset, -1 if none
    return dx >= 0 && dy >= 0 && dz >= 0 ? dx + 2 * dy + 4 * dz : dx <= 0 && dy <= 0 && dz <= 0 ? 7 - dx - 2 * dy - 4 * dz : -1;
}
// of u_c at neighbour k in 24 / h^2 (B_L u) at a node; of the pressure at neighbour k in 24 / h^2
// component c of (B_L^T p)
constexpr int div_coef(int k, int c) {
    int v = 0;
    for (int s = 0; s < 6; ++s)
        for (int a = 0; a < 4; ++a)
            for (int b = 0; b < 4; ++b)
                if (nbr_of(s, a, b) == k) v += grad(s, b, c);
    return v;
}
constexpr int grad_coef(int k, int c) {
    int v = 0;
    for (int s = 0; s < 6; ++s)
        for (int a = 0; a < 4; ++a)
            for (int b = 0; b < 4; ++b)
                if (nbr_of(s, a, b) == k) v += grad(s, a, c);
    return v;
}

// Both run one wavefront per 62 nodes of a lattice row, marching a chunk of layers: a lane holds the
// column x, the wavefront loads the rows y-1, y, y+1 of a layer once, one step ahead, and adds
// them to the sums of the three layers they are part of; the columns x-1 and x+1 come from the
// neighbour lanes by two DPP exchanges of the finished sums (the outer two lanes only feed
// them).  A workgroup is 4 rows, an XCD a slab of layers.  Bound by memory (129^3: 68 and 106 MB).
// Measured at 129^3: divergence 46 us with one thread per node, 45 loads and 144 products over
// the simplices, 32 with a row per wavefront and layer (21 loads), 27 marching; gradient
// with the interpolation of the pressure into a fine vector before it 37 us, 34 with the
// interpolation in the loads; 257^3 with W^-1 applied: 710 -> 357 and 660 -> 300 us (the fill and
// the elementwise products that went included).  Chunks of 8 to 32 layers measure alike.
constexpr int RX = 62, RY = NT / 64;
struct RowGrid {
    int gx, gy, gz, zc;
};
RowGrid row_grid(int n) {
    RowGrid g;
    g.gx = (n + RX) / RX;
    g.gy = (n + RY) / RY;
    g.zc = 32;
    while (g.zc > 2 && (int64_t)g.gx * g.gy * ((n + g.zc) / g.zc) < 2048) g.zc /= 2;
    g.gz = (n + g.zc) / g.zc;
    return g;
}
struct RowTile {
    int x, y, z0, z1, lane;
};
__device__ __forceinline__ RowTile row_tile(int n, const RowGrid& g) {
    const int cols = g.gx * g.gy, lin = tile_lin(cols, g.gz), bz = lin / cols, bc = lin - bz * cols;
    RowTile r;
    r.lane = threadIdx.x & 63;
    r.x = (bc % g.gx) * RX - 1 + r.lane;
    r.y = (bc / g.gx) * RY + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    r.z0 = bz * g.zc;
    r.z1 = min(r.z0 + g.zc - 1, n);
    return r;
}
// acc[0], acc[1], acc[2]: a lane's contributions to its right neighbour, itself and its left one
__device__ __forceinline__ double row_sum(const double (&acc)[3]) {
    const double l = shr1_row(acc[0]), r = shl1_row(acc[2]);
    return acc[1] + (l + r);
}

// q_v = -(B_L (s u))_v on every fine node, s elementwise (1 if null); velocity boundary values
// count as zero
template <bool SCALED>
__global__ void __launch_bounds__(NT)
k_div_fine(int n, const RowGrid g, const double* __restrict__ u, const double* __restrict__ s, double* __restrict__ q) {
    const RowTile p = row_tile(n, g);
    if (p.y > n) return;
    const int n1 = n + 1;
    const int64_t layer = (int64_t)n1 * n1, N = layer * n1;
    const uint32_t lbytes = (uint32_t)(layer * sizeof(double));
    const bool xin = p.x > 0 && p.x < n;
    uint32_t at[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) at[j] = xin && p.y + j > 1 && p.y + j <= n ? (uint32_t)(p.x + n1 * (p.y + j - 1)) * 8u : kOut;
    const uint32_t at_q = p.lane >= 1 && p.lane <= RX && p.x <= n ? (uint32_t)(p.x + n1 * p.y) * 8u : kOut;
    struct Rows {
        double v[3][3], s[SCALED ? 3 : 1][SCALED ? 3 : 1];
    };
    auto load = [&](int Z, Rows& r) {
        const bool zin = Z > 0 && Z < n && Z <= p.z1 + 1;
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                r.v[j][c] = bload<double>(layer_of(u + c * N + Z * layer, zin, lbytes), at[j]);
                if constexpr (SCALED) r.s[j][c] = bload<double>(layer_of(s + c * N + Z * layer, zin, lbytes), at[j]);
            }
    };
    const double h = 1.0 / n, w = h * h / 24.0;
    double acc[3][3] = {};  // of layers Z-1, Z, Z+1
    auto step = [&](int Z, const Rows& cur, Rows& nxt) {
        load(Z + 1, nxt);
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                double v = cur.v[j][c];
                if constexpr (SCALED) v *= cur.s[j][c];
#pragma unroll
                for (int dz = -1; dz <= 1; ++dz)
#pragma unroll
                    for (int dx = -1; dx <= 1; ++dx) {
                        // offset from the output node to the value: layer Z - dz
                        const int k = nbr_index(dx, j - 1, dz);
                        if (k >= 0 && div_coef(k, c) != 0)
                            acc[1 - dz][1 + dx] = fma((double)div_coef(k, c), v, acc[1 - dz][1 + dx]);
                    }
            }
        const double t = row_sum(acc[0]);
        bstore<double>(layer_of(q + (Z - 1) * layer, Z - 1 >= p.z0 && Z - 1 <= p.z1, lbytes), at_q, -w * t);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            acc[0][d] = acc[1][d];
            acc[1][d] = acc[2][d];
            acc[2][d] = 0.0;
        }
    };
    // two register sets in turn: a copy from one to the other would wait for its loads
    Rows even, odd;
    load(p.z0 - 1, even);
    for (int Z = p.z0 - 1; Z <= p.z1 + 1; Z += 2) {
        step(Z, even, odd);
        step(Z + 1, odd, even);
    }
}

// out = s (in - B_L^T (P pc)) on interior fine nodes (s = 1, in = 0 if null); on boundary nodes
// out = in.  pc: pressure on the level with n/2 cells; in may be out.
template <bool SCALED>
__global__ void __launch_bounds__(NT)
k_grad_fine(int n, const RowGrid g, const double* __restrict__ pc, const double* in, const double* __restrict__ s,
            double* out) {
    const RowTile p = row_tile(n, g);
    if (p.y > n) return;
    const int n1 = n + 1, c1 = n / 2 + 1;
    const int64_t layer = (int64_t)n1 * n1, N = layer * n1, clayer = (int64_t)c1 * c1;
    const uint32_t lbytes = (uint32_t)(layer * sizeof(double)), cbytes = (uint32_t)(clayer * sizeof(double));
    const bool xin = p.x >= 0 && p.x <= n;
    uint32_t lo[3], hi[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const int Y = p.y + j - 1;
        const bool ok = xin && Y >= 0 && Y <= n;
        lo[j] = ok ? (uint32_t)((p.x >> 1) + c1 * (Y >> 1)) * 8u : kOut;
        hi[j] = ok ? (uint32_t)(((p.x + 1) >> 1) + c1 * ((Y + 1) >> 1)) * 8u : kOut;
    }
    const uint32_t at = p.lane >= 1 && p.lane <= RX && p.x <= n ? (uint32_t)(p.x + n1 * p.y) * 8u : kOut;
    const bool inner = p.x > 0 && p.y > 0 && p.x < n && p.y < n;
    struct Rows {
        double lo[3], hi[3];
    };
    auto load = [&](int Z, Rows& r) {
        const bool zin = Z >= 0 && Z <= n && Z <= p.z1 + 1;
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            r.lo[j] = bload<double>(layer_of(pc + (Z >> 1) * clayer, zin, cbytes), lo[j]);
            r.hi[j] = bload<double>(layer_of(pc + ((Z + 1) >> 1) * clayer, zin, cbytes), hi[j]);
        }
    };
    struct Own {
        double in[3], s[SCALED ? 3 : 1];
    };
    auto load_own = [&](int z, Own& o) {
        const bool zin = z >= p.z0 && z <= p.z1;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            o.in[c] = bload<double>(layer_of(in + c * N + z * layer, zin && in, lbytes), at);
            if constexpr (SCALED) o.s[c] = bload<double>(layer_of(s + c * N + z * layer, zin, lbytes), at);
        }
    };
    const double h = 1.0 / n, w = h * h / 24.0;
    double acc[3][3][3] = {};  // of layers Z-1, Z, Z+1 and component c
    auto step = [&](int Z, const Rows& cur, const Own& own, Rows& nxt, Own& own_n) {
        load(Z + 1, nxt);
        load_own(Z, own_n);
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const double v = 0.5 * (cur.lo[j] + cur.hi[j]);
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int dz = -1; dz <= 1; ++dz)
#pragma unroll
                    for (int dx = -1; dx <= 1; ++dx) {
                        const int k = nbr_index(dx, j - 1, dz);
                        if (k >= 0 && grad_coef(k, c) != 0)
                            acc[1 - dz][c][1 + dx] = fma((double)grad_coef(k, c), v, acc[1 - dz][c][1 + dx]);
                    }
        }
        const int z = Z - 1;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double t = row_sum(acc[0][c]);
            double v = own.in[c] - w * t;
            if constexpr (SCALED) v *= own.s[c];
            bstore<double>(layer_of(out + c * N + z * layer, z >= p.z0 && z <= p.z1, lbytes), at,
                           inner && z > 0 && z < n ? v : own.in[c]);
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                acc[0][c][d] = acc[1][c][d];
                acc[1][c][d] = acc[2][c][d];
                acc[2][c][d] = 0.0;
            }
        }
    };
    Rows even, odd;
    Own own_e, own_o;
    load(p.z0 - 1, even);
    load_own(p.z0 - 2, own_e);
    for (int Z = p.z0 - 1; Z <= p.z1 + 1; Z += 2) {
        step(Z, even, own_e, odd, own_o);
        step(Z + 1, odd, own_o, even, own_e);
    }
}

// m_L(v) = h^3/24 sum_{d containing v} 1/nu_d on every fine node
__global__ void __launch_bounds__(NT)
k_mass_fine(int n, const double* __restrict__ nu, double* __restrict__ mf) {
    const int64_t n1 = n + 1, N = n1 * n1 * n1;
    const int64_t p = blockIdx.x * (int64_t)NT + threadIdx.x;
    if (p >= N) return;
    int x, y, z;
    node_xyz(p, n, x, y, z);
    const int64_t cells = (int64_t)n * n * n;
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        int64_t cell;
        if (!cell_of(n, x, y, z, k, cell)) continue;
#pragma unroll
        for (int s = 0; s < 6; ++s)
#pragma unroll
            for (int a = 0; a < 4; ++a)
                if (path_corner(s, a) == k) acc += 1.0 / nu[elem_slot(s, cell, cells)];
    }
    const double h = 1.0 / n;
    mf[p] = (h * h * h / 24.0) * acc;
}

// out = P^T qf over every node of the coarse level (nc cells), boundary included
__global__ void __launch_bounds__(NT)
k_restrict_all(int nc, const double* __restrict__ qf, double* __restrict__ out) {
    const int64_t nc1 = nc + 1, Nc = nc1 * nc1 * nc1;
    const int nf = 2 * nc;
    const int64_t nf1 = nf + 1;
    const int64_t p = blockIdx.x * (int64_t)NT + threadIdx.x;
    if (p >= Nc) return;
    int x, y, z;
    node_xyz(p, nc, x, y, z);
    const int X = 2 * x, Y = 2 * y, Z = 2 * z;
    double half = 0.0;
#pragma unroll
    for (int m = 1; m < 8; ++m) {
        const int dx = m & 1, dy = (m >> 1) & 1, dz = m >> 2;
#pragma unroll
        for (int sg = -1; sg <= 1; sg += 2) {
            const int qx = X + sg * dx, qy = Y + sg * dy, qz = Z + sg * dz;
            if (qx >= 0 && qy >= 0 && qz >= 0 && qx <= nf && qy <= nf && qz <= nf)
                half += qf[qx + nf1 * (qy + nf1 * (int64_t)qz)];
        }
    }
    out[p] = qf[X + nf1 * (Y + nf1 * (int64_t)Z)] + 0.5 * half;
}

// pf = P pc (ADD: pf += P pc) on every node of the fine level (nf cells), boundary included
template <bool ADD>
__global__ void __launch_bounds__(NT)
k_prolong_all(int nf, const double* __restrict__ pc, double* __restrict__ pf) {
    const int nc = nf / 2;
    const int64_t nc1 = nc + 1;
    const int64_t Nf = (int64_t)(nf + 1) * (nf + 1) * (nf + 1);
    const int64_t p = blockIdx.x * (int64_t)NT + threadIdx.x;
    if (p >= Nf) return;
    int x, y, z;
    node_xyz(p, nf, x, y, z);
    const int dx = x & 1, dy = y & 1, dz = z & 1;
    const int64_t lo = ((x - dx) >> 1) + nc1 * (((y - dy) >> 1) + nc1 * (int64_t)((z - dz) >> 1));
    const int64_t hi = ((x + dx) >> 1) + nc1 * (((y + dy) >> 1) + nc1 * (int64_t)((z + dz) >> 1));
    const double v = (dx | dy | dz) ? 0.5 * (pc[lo] + pc[hi]) : pc[lo];
    pf[p] = ADD ? pf[p] + v : v;
}

__global__ void __launch_bounds__(NT)
k_div_elementwise(int64_t n, const double* __restrict__ num, const double* __restrict__ den,
                  double* __restrict__ out) {
    const int64_t stride = (int64_t)gridDim.x * NT;
    for (int64_t i = blockIdx.x * (int64_t)NT + threadIdx.x; i < n; i += stride) out[i] = num[i] / den[i];
}

// Colour (x mod 3) + 3 (y mod 3) + 9 (z mod 3) of the nodes of a level with n cells per
// axis.  mode 0: out = indicator of the colour; mode 1: out = src on the colour's nodes
// (others untouched).
__global__ void __launch_bounds__(NT)
k_colour(int n, int colour, int mode, const double* __restrict__ src, double* __restrict__ out) {
    const int64_t n1 = n + 1, N = n1 * n1 * n1;
    const int64_t stride = (int64_t)gridDim.x * NT;
    for (int64_t p = blockIdx.x * (int64_t)NT + threadIdx.x; p < N; p += stride) {
        int x, y, z;
        node_coords(p, n, x, y, z);
        const bool on = (x % 3) + 3 * (y % 3) + 9 * (z % 3) == colour;
        if (mode == 0)
            out[p] = on ? 1.0 : 0.0;
        else if (on)
            out[p] = src[p];
    }
}

// y += sign * coef[0] * x with the coefficient read from device memory
__global__ void __launch_bounds__(NT)
k_axpy_dev(int64_t n, const double* __restrict__ coef, double sign, const double* __restrict__ x,
           double* __restrict__ y) {
    const double a = sign * coef[0];
    const int64_t stride = (int64_t)gridDim.x * NT;
    for (int64_t i = blockIdx.x * (int64_t)NT + threadIdx.x; i < n; i += stride) y[i] += a * x[i];
}

// Classical Gram-Schmidt against nv contiguous vectors V_i = V + i * ld (the FGMRES
// basis): one pass over w and the basis for all the dot products, one for the update.
// A workgroup owns GS_CHUNK consecutive entries; each thread keeps its GS_PER entries of
// w in registers while the workgroup walks the basis, so w is read once.  The dots of
// every workgroup are reduced in a fixed order (wavefront shuffles, then LDS), and the
// partials of all workgroups by k_gs_sum, so the results are bitwise reproducible.
constexpr int GS_PER = 8;
constexpr int GS_CHUNK = NT * GS_PER;

__device__ __forceinline__ double gs_wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    return v;
}

// partial[i * gridDim.x + block] = sum over the block's entries of w V_i (i < nv), and
// partial[nv * gridDim.x + block] = sum of w^2; a basis stored in FP32 is widened on
// the fly (the products and sums stay FP64)
template <typename VT>
__global__ void __launch_bounds__(NT)
k_gs_dots(int64_t n, const double* __restrict__ w, const VT* __restrict__ V, int64_t ld, int nv,
          double* __restrict__ partial) {
    __shared__ double red[NT / 64];
    const int64_t base = (int64_t)blockIdx.x * GS_CHUNK + threadIdx.x;
    double wv[GS_PER];
#pragma unroll
    for (int m = 0; m < GS_PER; ++m) {
        const int64_t j = base + (int64_t)m * NT;
        wv[m] = j < n ? w[j] : 0.0;
    }
    for (int i = 0; i <= nv; ++i) {
        double acc = 0.0;
        if (i < nv) {
            const VT* v = V + (int64_t)i * ld;
#pragma unroll
            for (int m = 0; m < GS_PER; ++m) {
                const int64_t j = base + (int64_t)m * NT;
                acc += wv[m] * (j < n ? (double)v[j] : 0.0);
            }
        } else {
#pragma unroll
            for (int m = 0; m < GS_PER; ++m) acc += wv[m] * wv[m];
        }
        acc = gs_wave_sum(acc);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
        __syncthreads();
        if (threadIdx.x == 0) {
            double t = 0.0;
            for (int q = 0; q < NT / 64; ++q) t += red[q];
            partial[(int64_t)i * gridDim.x + blockIdx.x] = t;
        }
        __syncthreads();
    }
}

// out[i] = sum over the nb partials of row i (one workgroup per row, fixed order)
__global__ void __launch_bounds__(NT)
k_gs_sum(const double* __restrict__ partial, int nb, double* __restrict__ out) {
    __shared__ double red[NT / 64];
    const double* row = partial + (int64_t)blockIdx.x * nb;
    double acc = 0.0;
    for (int b = threadIdx.x; b < nb; b += NT) acc += row[b];
    acc = gs_wave_sum(acc);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int q = 0; q < NT / 64; ++q) t += red[q];
        out[blockIdx.x] = t;
    }
}

// w -= sum_i h[i] V_i (h on the device), and per workgroup the partial sum of the new w^2 (in the
// order of k_gs_dots: the pass of its own over w that this replaces gave the same bits)
__device__ __forceinline__ void gs_store_partial(double acc, double* __restrict__ partial) {
    __shared__ double red[NT / 64];
    acc = gs_wave_sum(acc);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int q = 0; q < NT / 64; ++q) t += red[q];
        partial[blockIdx.x] = t;
    }
}
__global__ void __launch_bounds__(NT)
k_gs_update(int64_t n, double* __restrict__ w, const double* __restrict__ V, int64_t ld, int nv,
            const double* __restrict__ h, double* __restrict__ partial) {
    const int64_t base = (int64_t)blockIdx.x * GS_CHUNK + threadIdx.x;
    double a[GS_PER] = {};
#pragma unroll 2
    for (int i = 0; i < nv; ++i) {
        const double* v = V + (int64_t)i * ld;
        const double hi = h[i];
#pragma unroll
        for (int m = 0; m < GS_PER; ++m) {
            const int64_t j = base + (int64_t)m * NT;
            a[m] += hi * (j < n ? v[j] : 0.0);
        }
    }
    double acc = 0.0;
#pragma unroll
    for (int m = 0; m < GS_PER; ++m) {
        const int64_t j = base + (int64_t)m * NT;
        if (j < n) {
            const double t = w[j] - a[m];
            w[j] = t;
            acc += t * t;
        }
    }
    gs_store_partial(acc, partial);
}

// The same two passes over an FP32 basis, four consecutive entries per lane and load
// (the basis vectors start at 16-byte aligned offsets, ld a multiple of 4): a wavefront
// then keeps as many bytes in flight per basis vector as the FP64 passes (with one
// 4-byte load per entry the passes ran at 3.8 TB/s against 5.3 for the FP64 basis).
// The dot pass owns GS_CHUNK_F32 = 2 GS_CHUNK entries per workgroup (gs_blocks_f32).
constexpr int GS_QUADS = 4;                   // float4 loads per lane and basis vector
constexpr int GS_CHUNK_F32 = NT * 4 * GS_QUADS;

__global__ void __launch_bounds__(NT)
k_gs_dots_f32(int64_t n, const double* __restrict__ w, const float* __restrict__ V, int64_t ld, int nv,
              double* __restrict__ partial) {
    __shared__ double red[NT / 64];
    const int64_t base = (int64_t)blockIdx.x * GS_CHUNK_F32 + 4 * threadIdx.x;
    double wv[4 * GS_QUADS];
#pragma unroll
    for (int q = 0; q < GS_QUADS; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int64_t j = base + (int64_t)q * 4 * NT + e;
            wv[4 * q + e] = j < n ? w[j] : 0.0;
        }
    for (int i = 0; i <= nv; ++i) {
        double acc = 0.0;
        if (i < nv) {
            const float* v = V + (int64_t)i * ld;
            float4 vv[GS_QUADS];
#pragma unroll
            for (int q = 0; q < GS_QUADS; ++q) {
                // the quad starts inside the padded vector (ld >= n, a multiple of 4)
                const int64_t j = base + (int64_t)q * 4 * NT;
                vv[q] = j < n ? *reinterpret_cast<const float4*>(v + j) : float4{0.0f, 0.0f, 0.0f, 0.0f};
            }
#pragma unroll
            for (int q = 0; q < GS_QUADS; ++q) {
                const int64_t j = base + (int64_t)q * 4 * NT;
                const float f[4] = {vv[q].x, vv[q].y, vv[q].z, vv[q].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) acc += wv[4 * q + e] * (j + e < n ? (double)f[e] : 0.0);
            }
        } else {
#pragma unroll
            for (int m = 0; m < 4 * GS_QUADS; ++m) acc += wv[m] * wv[m];
        }
        acc = gs_wave_sum(acc);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
        __syncthreads();
        if (threadIdx.x == 0) {
            double t = 0.0;
            for (int q = 0; q < NT / 64; ++q) t += red[q];
            partial[(int64_t)i * gridDim.x + blockIdx.x] = t;
        }
        __syncthreads();
    }
}

// w -= sum_i h[i] V_i over four consecutive entries per lane, the basis loads of four
// vectors issued before their products are summed (in the order of i, as above)
__global__ void __launch_bounds__(NT)
k_gs_update_f32(int64_t n, double* __restrict__ w, const float* __restrict__ V, int64_t ld, int nv,
                const double* __restrict__ h, double* __restrict__ partial) {
    const int64_t stride = (int64_t)gridDim.x * NT;
    double acc = 0.0;
    for (int64_t j = 4 * (blockIdx.x * (int64_t)NT + threadIdx.x); j < n; j += 4 * stride) {
        double a[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
        for (int i = 0; i < nv; ++i) {
            const float4 vv = *reinterpret_cast<const float4*>(V + (int64_t)i * ld + j);
            const double hi = h[i];
            a[0] += hi * (double)vv.x;
            a[1] += hi * (double)vv.y;
            a[2] += hi * (double)vv.z;
            a[3] += hi * (double)vv.w;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (j + e < n) {
                const double t = w[j + e] - a[e];
                w[j + e] = t;
                acc += t * t;
            }
    }
    gs_store_partial(acc, partial);
}

// y = a x rounded to FP32 (a new FP32 basis vector)
__global__ void __launch_bounds__(NT)
k_scale_to_f32(int64_t n, double a, const double* __restrict__ x, float* __restrict__ y) {
    const int64_t stride = (int64_t)gridDim.x * NT;
    for (int64_t j = blockIdx.x * (int64_t)NT + threadIdx.x; j < n; j += stride) y[j] = (float)(a * x[j]);
}

unsigned grid_for(int64_t n) { return (unsigned)((n + NT - 1) / NT); }
unsigned grid_stride(int64_t n) {
    const int64_t g = (n + NT - 1) / NT;
    return (unsigned)(g < 4096 ? (g > 0 ? g : 1) : 4096);
}

}  // namespace

hipError_t launch_stokes_div_fine(int n, const double* u, const double* s, double* q, hipStream_t st) {
    if (!u || !q || n < 2) return hipErrorInvalidValue;
    const RowGrid g = row_grid(n);
    const dim3 grid((unsigned)((int64_t)g.gx * g.gy * g.gz));
    if (s)
        hipLaunchKernelGGL(k_div_fine<true>, grid, dim3(NT), 0, st, n, g, u, s, q);
    else
        hipLaunchKernelGGL(k_div_fine<false>, grid, dim3(NT), 0, st, n, g, u, s, q);
    return hipGetLastError();
}
hipError_t launch_stokes_grad(int n, const double* pc, const double* in, const double* s, double* out, hipStream_t st) {
    if (!pc || !out || n < 2) return hipErrorInvalidValue;
    const RowGrid g = row_grid(n);
    const dim3 grid((unsigned)((int64_t)g.gx * g.gy * g.gz));
    if (s)
        hipLaunchKernelGGL(k_grad_fine<true>, grid, dim3(NT), 0, st, n, g, pc, in, s, out);
    else
        hipLaunchKernelGGL(k_grad_fine<false>, grid, dim3(NT), 0, st, n, g, pc, in, s, out);
    return hipGetLastError();
}
hipError_t launch_stokes_mass_fine(int n, const double* nu, double* mf, hipStream_t st) {
    if (!nu || !mf || n < 2) return hipErrorInvalidValue;
    const int64_t N = (int64_t)(n + 1) * (n + 1) * (n + 1);
    hipLaunchKernelGGL(k_mass_fine, dim3(grid_for(N)), dim3(NT), 0, st, n, nu, mf);
    return hipGetLastError();
}
hipError_t launch_restrict_all(int n_coarse, const double* qf, double* out, hipStream_t st) {
    if (!qf || !out || n_coarse < 1) return hipErrorInvalidValue;
    const int64_t N = (int64_t)(n_coarse + 1) * (n_coarse + 1) * (n_coarse + 1);
    hipLaunchKernelGGL(k_restrict_all, dim3(grid_for(N)), dim3(NT), 0, st, n_coarse, qf, out);
    return hipGetLastError();
}
hipError_t launch_prolong_all(int n_fine, const double* pc, double* pf, hipStream_t st) {
    if (!pc || !pf || n_fine < 2) return hipErrorInvalidValue;
    const int64_t N = (int64_t)(n_fine + 1) * (n_fine + 1) * (n_fine + 1);
    hipLaunchKernelGGL(k_prolong_all<false>, dim3(grid_for(N)), dim3(NT), 0, st, n_fine, pc, pf);
    return hipGetLastError();
}
hipError_t launch_prolong_all_add(int n_fine, const double* pc, double* pf, hipStream_t st) {
    if (!pc || !pf || n_fine < 2) return hipErrorInvalidValue;
    const int64_t N = (int64_t)(n_fine + 1) * (n_fine + 1) * (n_fine + 1);
    hipLaunchKernelGGL(k_prolong_all<true>, dim3(grid_for(N)), dim3(NT), 0, st, n_fine, pc, pf);
    return hipGetLastError();
}
hipError_t launch_div_elementwise(int64_t n, const double* num, const double* den, double* out,
                                  hipStream_t st) {
    if (!num || !den || !out) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_div_elementwise, dim3(grid_stride(n)), dim3(NT), 0, st, n, num, den, out);
    return hipGetLastError();
}

hipError_t launch_colour(int n, int colour, int mode, const double* src, double* out, hipStream_t st) {
    if (n < 1 || colour < 0 || colour > 26 || !out || (mode == 1 && !src)) return hipErrorInvalidValue;
    const int64_t N = (int64_t)(n + 1) * (n + 1) * (n + 1);
    hipLaunchKernelGGL(k_colour, dim3(grid_stride(N)), dim3(NT), 0, st, n, colour, mode, src, out);
    return hipGetLastError();
}
int gs_blocks(int64_t n) { return (int)((n + GS_CHUNK - 1) / GS_CHUNK); }
int gs_blocks_f32(int64_t n) { return (int)((n + GS_CHUNK_F32 - 1) / GS_CHUNK_F32); }
template <typename VT>
hipError_t launch_gs_dots(int64_t n, const double* w, const VT* V, int64_t ld, int nv,
                          double* partial, hipStream_t st) {
    if (!w || !V || !partial || n <= 0 || nv < 0) return hipErrorInvalidValue;
    if constexpr (sizeof(VT) == 4) {
        // quad loads: leading dimension a multiple of 4 covering n, 16-byte aligned base
        if ((ld & 3) || ld < n || (reinterpret_cast<uintptr_t>(V) & 15)) return hipErrorInvalidValue;
        hipLaunchKernelGGL(k_gs_dots_f32, dim3((unsigned)gs_blocks_f32(n)), dim3(NT), 0, st, n, w, V, ld, nv,
                           partial);
    } else {
        hipLaunchKernelGGL(k_gs_dots<VT>, dim3((unsigned)gs_blocks(n)), dim3(NT), 0, st, n, w, V, ld, nv,
                           partial);
    }
    return hipGetLastError();
}
template hipError_t launch_gs_dots<double>(int64_t, const double*, const double*, int64_t, int, double*,
                                           hipStream_t);
template hipError_t launch_gs_dots<float>(int64_t, const double*, const float*, int64_t, int, double*,
                                          hipStream_t);
hipError_t launch_gs_sum(const double* partial, int nb, int rows, double* out, hipStream_t st) {
    if (!partial || !out || nb <= 0 || rows <= 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_gs_sum, dim3((unsigned)rows), dim3(NT), 0, st, partial, nb, out);
    return hipGetLastError();
}
template <typename VT>
hipError_t launch_gs_update(int64_t n, double* w, const VT* V, int64_t ld, int nv, const double* h, double* partial,
                            hipStream_t st) {
    if (!w || !V || !h || !partial || n <= 0 || nv <= 0) return hipErrorInvalidValue;
    if constexpr (sizeof(VT) == 4) {
        if ((ld & 3) || ld < n || (reinterpret_cast<uintptr_t>(V) & 15)) return hipErrorInvalidValue;
        hipLaunchKernelGGL(k_gs_update_f32, dim3((unsigned)gs_blocks_f32(n)), dim3(NT), 0, st, n, w, V, ld, nv, h,
                           partial);
    } else {
        hipLaunchKernelGGL(k_gs_update, dim3((unsigned)gs_blocks(n)), dim3(NT), 0, st, n, w, V, ld, nv, h, partial);
    }
    return hipGetLastError();
}
template hipError_t launch_gs_update<double>(int64_t, double*, const double*, int64_t, int, const double*, double*,
                                             hipStream_t);
template hipError_t launch_gs_update<float>(int64_t, double*, const float*, int64_t, int, const double*, double*,
                                            hipStream_t);
hipError_t launch_scale_to_f32(int64_t n, double a, const double* x, float* y, hipStream_t st) {
    if (!x || !y || n <= 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_scale_to_f32, dim3(grid_stride(n)), dim3(NT), 0, st, n, a, x, y);
    return hipGetLastError();
}
hipError_t launch_axpy_dev(int64_t n, const double* coef, double sign, const double* x, double* y,
                           hipStream_t st) {
    if (!coef || !x || !y) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_axpy_dev, dim3(grid_stride(n)), dim3(NT), 0, st, n, coef, sign, x, y);
    return hipGetLastError();
}

}  // namespace agca
