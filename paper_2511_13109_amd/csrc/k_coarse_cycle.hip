// The coarse end of the V-cycle (Section 2.1's multigrid cycle) in one workgroup.
//
// On the small levels a pass is a few thousand rows of work, and as separate launches every
// pass costs a kernel's start and drain on the GPU (2.5-5 us) whatever its size.  Here one
// workgroup runs the whole down and up sweep of levels K..1 plus the level-0 solve with
// workgroup barriers between the passes.  A thread owns fixed rows (node, component) of
// every level: their right-hand side, inverse diagonal, iterate and previous iterate stay in
// its registers, and only the iterate's values that neighbours read (two buffers per level)
// are in LDS.  The operator's rows are read once: the top level's into registers (scalar: the
// six weights of the seven-point form, k_scalar.hip; vector: of the 15-point stencil the 37
// entries that are not identically zero, formed from the coefficient), the lower levels' into LDS.
// (A component couples with itself along lattice axes only: unit_entry, kuhn.h, is the path
// Laplacian plus the product of two gradient components, which for equal components is
// non-zero only across a step along that axis.)
//
// K: scalar hierarchies up to 17^3 nodes (K = 3), vector ones up to 9^3 (K = 2: the 1029 rows of
// 37 entries are what the registers of 512 threads hold; the five rows beyond stay in LDS); the
// whole cycle where that is the finest level.  The vector rows are formed here, from the 24 KB
// of coefficients of a 9^3 level: read as an assembled stencil they are 0.8 MB (FP64), after
// fine levels that push them out of the caches more than one compute unit reads in the time
// of the launches it saves (FP32 17^3 cycle from cold caches 67 us, 59 with launches for the 9^3
// level, 52 this way; FP64 70, 73 and 62).  With caches flushed between cycles (1 GB written; us with K = 3 / 2 / 1 / one
// launch per pass above 5^3 or 9^3): scalar 17^3 FP64 23.0 / 26.6 / 40.7 / 42.8, FP32 19.1 / 25.5 / 39.0 / 38.4; 33^3
// FP64 41.0 / 44.8 / 59.1 / 63.2, FP32 35.8 / 42.9 / 56.4 / 55.9; vector from K = 2 on: 9^3 FP64 27.4 / 45.4 / 53.6,
// 17^3 64.0 / 72.5 / 80.8, FP32 52.8 / 59.1 / 62.0.
// A pass is bound by the LDS reads of the neighbours (9^3 vector FP64: 37 per row, about
// 1 us) and the barrier.  Whole cycles, Chebyshev (2, 2), before (one launch per pass above
// 5^3 / 9^3) and now: scalar 9^3 27 -> 5.4 us, 17^3 FP64 36 -> 16.7, FP32 32 -> 12.5; vector
// 9^3 FP64 47 -> 21, FP32 36 -> 15.5, 17^3 72 -> 56 and 56 -> 45.
#include <hip/hip_runtime.h>

#include "internal.h"
#include "kuhn.h"
#include "level_ops.h"

namespace agca {
namespace {

// threads: 1024 of 128 registers, or 512 of 256 where a thread's rows take more than half of
// 128 (FP64, and the 37 entries of a vector row).  17^3 scalar cycle: FP64 23.0 us with 1024
// threads, 17.4 with 512; FP32 13.7 and 14.6.
constexpr int ct(int nc, size_t elem) { return nc == 1 && elem == 4 ? 1024 : 512; }
constexpr int row_regs(int nc, size_t elem) { return nc == 1 ? 4096 / ct(nc, elem) : 2; }

constexpr int kReads = 8;  // a vector row's neighbour reads in flight (all 37: the registers of a row)
constexpr int max_level(int nc) { return nc == 1 ? 3 : 2; }

constexpr int lvl_n(int l) { return 2 << l; }
constexpr int lvl_nodes(int l) { return (lvl_n(l) + 1) * (lvl_n(l) + 1) * (lvl_n(l) + 1); }
constexpr int lvl_free(int l) { return (lvl_n(l) - 1) * (lvl_n(l) - 1) * (lvl_n(l) - 1); }
// rows of a level and rows per thread
constexpr int lvl_rows(int nc, int l) { return nc * lvl_free(l); }
constexpr int lvl_slots(int nc, size_t elem, int l) {
    return (lvl_rows(nc, l) + ct(nc, elem) - 1) / ct(nc, elem);
}
// operator entries per row
constexpr int row_terms(int nc) { return nc == 1 ? 6 : 37; }
// rows whose operator entries live in LDS: all rows of the levels below K, and the rows of
// level K beyond what the registers hold
constexpr int lds_rows(int nc, size_t elem, int l, int K) {
    const int held = l < K ? 0 : row_regs(nc, elem) * ct(nc, elem);
    return lvl_rows(nc, l) > held ? lvl_rows(nc, l) - held : 0;
}
constexpr int x_offset(int nc, int l) {  // first of a level's two iterate buffers
    int o = 0;
    for (int j = 0; j < l; ++j) o += 2 * nc * lvl_nodes(j);
    return o;
}
constexpr int s_offset(int nc, size_t elem, int l, int K) {
    int o = x_offset(nc, K + 1);
    for (int j = 1; j < l; ++j) o += row_terms(nc) * lds_rows(nc, elem, j, K);
    return o;
}
constexpr int lds_values(int nc, size_t elem, int K) { return s_offset(nc, elem, K + 1, K); }

template <int NC, int LV>
__device__ __forceinline__ int row_addr(int row) {  // slot c N + p of a row in a level vector
    constexpr int n = lvl_n(LV), m = n - 1, I = lvl_free(LV);
    const int c = row / I, i = row - c * I;
    const int z = i / (m * m), r = i - z * m * m, y = r / m, x = r - y * m;
    return c * lvl_nodes(LV) + (x + 1) + (n + 1) * ((y + 1) + (n + 1) * (z + 1));
}

// a row's address as an unknown value: what is derived from it for one transfer is computed
// there, not kept in registers from the first use on
__device__ __forceinline__ int reread(int addr) {
    asm volatile("" : "+v"(addr));
    return addr;
}

// neighbour index (kuhn.h) of the q-th of the seven axis neighbours: the node, +x, +y, +z, -x, -y, -z
constexpr int axis_nbr(int q) { return q == 0 ? 0 : q < 4 ? 1 << (q - 1) : 7 + (1 << (q - 4)); }
// term t of a vector row of component c: neighbour index, and component relative to c
constexpr int term_nbr(int t) { return t < 7 ? axis_nbr(t) : (t - 7) % kStencilPoints; }
constexpr int term_comp(int t) { return t < 7 ? 0 : 1 + (t - 7) / kStencilPoints; }

// term of neighbour k (kuhn.h) and component d of a row of component c
constexpr int term_of(int k, int d, int c) {
    const int rel = (d - c + 3) % 3;
    if (rel > 0) return 7 + (rel - 1) * kStencilPoints + k;
    for (int q = 0; q < 7; ++q)
        if (axis_nbr(q) == k) return q;
    return -1;
}

// the entries of the row (C, p) of the vector operator from the coefficient, in FP64: the
// assembly of k_stencil.hip, in its order
template <int C, int LV>
__device__ __forceinline__ void assemble_row(const double* __restrict__ nu, int p, double (&acc)[37]) {
    constexpr int n = lvl_n(LV), n1 = n + 1;
    const double scale = 1.0 / (6.0 * n);
    const int z = p / (n1 * n1), r = p - z * n1 * n1, y = r / n1, x = r - y * n1;
#pragma unroll
    for (int t = 0; t < 37; ++t) acc[t] = 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int cell = x - (k & 1) + n * (y - ((k >> 1) & 1) + n * (z - (k >> 2)));
#pragma unroll
        for (int s = 0; s < 6; ++s)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                if (path_corner(s, a) != k) continue;
                const double w = nu[elem_slot(s, cell, n * n * n)] * scale;
#pragma unroll
                for (int b = 0; b < 4; ++b)
#pragma unroll
                    for (int d = 0; d < 3; ++d)
                        if (unit_entry(s, C, a, d, b) != 0)
                            acc[term_of(nbr_of(s, a, b), d, C)] += w * (double)unit_entry(s, C, a, d, b);
            }
    }
}

// the entries of row (c, p): scalar, the weights of the edges to x-1, x+1, y-1, y+1, z-1, z+1;
// vector, the terms of the stencil row.  put(t, value) for each.
template <int NC, typename T, int LV, typename P>
__device__ __forceinline__ void load_row(const CoarseCycle<T>& a, int addr, const P& put) {
    constexpr unsigned n1 = lvl_n(LV) + 1, N = lvl_nodes(LV);
    if constexpr (NC == 1) {
#pragma unroll
        for (int t = 0; t < 6; ++t) {
            const unsigned ax = t >> 1, step = ax == 0 ? 1 : ax == 1 ? n1 : n1 * n1;
            put(t, a.wts[LV][ax * N + (unsigned)addr - ((t & 1) ? 0u : step)]);
        }
    } else {
        const int c = addr / (int)N, p = addr - c * (int)N;
        double e[37];
        if (c == 0)
            assemble_row<0, LV>(a.nu[LV], p, e);
        else if (c == 1)
            assemble_row<1, LV>(a.nu[LV], p, e);
        else
            assemble_row<2, LV>(a.nu[LV], p, e);
#pragma unroll
        for (int t = 0; t < row_terms(NC); ++t) put(t, T(e[t]));
    }
}

// A u at a row: u the level's iterate buffer in LDS (0 on the boundary), entry(t) the row's
template <int NC, typename T, int LV, typename E>
__device__ __forceinline__ T row_product(const T* u, int addr, const E& entry) {
    constexpr int n1 = lvl_n(LV) + 1, N = lvl_nodes(LV);
    // LDS instructions add non-negative offsets only: the reads are based at the lowest one
    constexpr int low = NC == 1 ? n1 * n1 : n1 * n1 + n1 + 1;
    T acc = T(0);
    if constexpr (NC == 1) {
        const T* ub = u + addr - low;
        const T c = ub[low];
#pragma unroll
        for (int t = 0; t < 6; ++t) {
            const int ax = t >> 1, step = ax == 0 ? 1 : ax == 1 ? n1 : n1 * n1;
            acc = fma(entry(t), c - ub[low + ((t & 1) ? step : -step)], acc);
        }
    } else {
        const int c = reread(addr) / N;
        int at[3] = {addr - low, addr - low + (c < 2 ? N : -2 * N), addr - low + (c < 1 ? 2 * N : -N)};
#pragma unroll
        for (int t = 0; t < row_terms(NC); ++t) {
            const int m = nbr_mask(term_nbr(t)), sg = nbr_sign(term_nbr(t));
            acc = fma(entry(t), u[at[term_comp(t)] + low + sg * ((m & 1) + n1 * (((m >> 1) & 1) + n1 * (m >> 2)))], acc);
            // the reads of some neighbours at a time: all in flight would not fit beside the
            // row's entries
            if (t % kReads == kReads - 1) asm volatile("" : "+v"(at[0]), "+v"(at[1]), "+v"(at[2]), "+v"(acc));
        }
    }
    return acc;
}

template <int NC, typename T, int K, int LV>
struct LevelCycle {
    static constexpr int SLOTS = lvl_slots(NC, sizeof(T), LV), ROWS = lvl_rows(NC, LV), VEC = NC * lvl_nodes(LV);
    static constexpr bool TOP = LV == K;
    static constexpr int CT = ct(NC, sizeof(T));
    // slots with their operator entries in registers
    static constexpr int REG = TOP ? (SLOTS < row_regs(NC, sizeof(T)) ? SLOTS : row_regs(NC, sizeof(T))) : 0;
    T w[REG > 0 ? REG : 1][row_terms(NC)];
    T b[SLOTS], d[SLOTS], cur[SLOTS], prv[SLOTS];
    int addr[SLOTS];

    static __device__ __forceinline__ bool has(int s) { return (int)threadIdx.x + s * CT < ROWS; }

    // the thread's rows; the operator rows that live in LDS are copied there
    __device__ __forceinline__ void init(const CoarseCycle<T>& a, T* lds) {
        const int tid = threadIdx.x;
        constexpr int LR = lds_rows(NC, sizeof(T), LV, K);
        if constexpr (LR > 0) {
            T* S = lds + s_offset(NC, sizeof(T), LV, K);
            for (int i = tid; i < LR; i += CT) {
                load_row<NC, T, LV>(a, row_addr<NC, LV>(i + (ROWS - LR)), [&](int t, T v) { S[t * LR + i] = v; });
            }
        }
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            // rows past the last repeat row 0; their results are never stored
            addr[s] = row_addr<NC, LV>(has(s) ? tid + s * CT : 0);
            d[s] = a.dinv[LV][addr[s]];
            b[s] = cur[s] = prv[s] = T(0);
            if (s < REG) load_row<NC, T, LV>(a, addr[s], [&](int t, T v) { w[s < REG ? s : 0][t] = v; });
        }
    }
    __device__ __forceinline__ T product(const T* lds, const T* u, int s) const {
        if (s < REG) return row_product<NC, T, LV>(u, addr[s], [&](int t) { return w[s < REG ? s : 0][t]; });
        constexpr int LR = lds_rows(NC, sizeof(T), LV, K) > 0 ? lds_rows(NC, sizeof(T), LV, K) : 1;
        const T* S = lds + s_offset(NC, sizeof(T), LV, K);
        const int i = min((int)threadIdx.x + s * CT - (ROWS - LR), LR - 1);
        return row_product<NC, T, LV>(u, addr[s], [&](int t) { return S[t * LR + i]; });
    }
    __device__ __forceinline__ void put(T* u) const {
#pragma unroll
        for (int s = 0; s < SLOTS; ++s)
            if (has(s)) u[addr[s]] = cur[s];
    }
    // x <- alpha x + gamma x_prev + omega D^-1 (b - A x), from buffer u into buffer v
    __device__ __forceinline__ void pass(T* lds, const T* u, T* v, bool cheb, const T (&c)[3]) {
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            if (!has(s)) continue;
            const T r = b[s] - product(lds, u, s);
            const T nx = fma(c[2] * d[s], r, cheb ? fma(c[1], prv[s], c[0] * cur[s]) : c[0] * cur[s]);
            prv[s] = cur[s];
            cur[s] = nx;
            // two scalar rows' reads in flight
            if constexpr (NC == 1 && SLOTS > 2)
                if (s % 2 == 1 && s + 1 < SLOTS)
                    asm volatile("" : "+v"(cur[s]), "+v"(addr[s + 1]), "+v"(addr[s + 2 < SLOTS ? s + 2 : s]));
        }
        put(v);
        __syncthreads();
    }
    // one cycle from zero for the right-hand side in b; on return cur holds the thread's rows
    // and the buffer returned holds the iterate
    template <typename Lower>
    __device__ __forceinline__ T* run(const CoarseCycle<T>& a, T* lds, Lower& lower) {
        T* u = lds + x_offset(NC, LV);
        T* v = u + VEC;
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            cur[s] = a.pre > 0 ? a.c[LV - 1][0][2] * d[s] * b[s] : T(0);
            prv[s] = T(0);
        }
        put(u);
        __syncthreads();
        for (int k = 1; k < a.pre; ++k) {
            pass(lds, u, v, a.cheb != 0, a.c[LV - 1][k]);
            T* t = u; u = v; v = t;
        }
        // residual into the free buffer, restricted by the rows' owners on the level below
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            if (!has(s)) continue;
            v[addr[s]] = b[s] - product(lds, u, s);
        }
        __syncthreads();
        lower.take(v);
        const T* e = lower.cycle(a, lds);
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            if (!has(s)) continue;
            constexpr int n1 = lvl_n(LV) + 1, N = lvl_nodes(LV), c1 = lvl_n(LV - 1) + 1, Nc = lvl_nodes(LV - 1);
            const int ad = reread(addr[s]), c = ad / N, p = ad - c * N;
            const int z = p / (n1 * n1), q = p - z * n1 * n1, y = q / n1, x = q - y * n1;
            const int lo = (x >> 1) + c1 * ((y >> 1) + c1 * (z >> 1));
            const int hi = ((x + 1) >> 1) + c1 * (((y + 1) >> 1) + c1 * ((z + 1) >> 1));
            cur[s] += T(0.5) * (e[c * Nc + lo] + e[c * Nc + hi]);
        }
        put(u);
        __syncthreads();
        for (int k = 0; k < a.post; ++k) {
            pass(lds, u, v, a.cheb != 0 && k > 0, a.c[LV - 1][k]);
            T* t = u; u = v; v = t;
        }
        return u;
    }
    // b <- P^T r at the thread's rows, r the residual buffer of level LV + 1
    __device__ __forceinline__ void restrict_from(const T* r) {
        constexpr int n1 = lvl_n(LV) + 1, N = lvl_nodes(LV), f1 = lvl_n(LV + 1) + 1, Nf = lvl_nodes(LV + 1);
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            if (!has(s)) continue;
            const int ad = reread(addr[s]), c = ad / N, p = ad - c * N;
            const int z = p / (n1 * n1), q = p - z * n1 * n1, y = q / n1, x = q - y * n1;
            const T* f = r + c * Nf + 2 * x + f1 * (2 * y + f1 * 2 * z);
            T half = T(0);
#pragma unroll
            for (int k = 1; k < 8; ++k) {
                const int off = (k & 1) + f1 * (((k >> 1) & 1) + f1 * (k >> 2));
                half += f[off] + f[-off];
            }
            b[s] = f[0] + T(0.5) * half;
        }
    }
};

// levels LV..0 as one object: the recursion's lower part
template <int NC, typename T, int K, int LV>
struct Levels {
    LevelCycle<NC, T, K, LV> top;
    Levels<NC, T, K, LV - 1> lower;
    __device__ __forceinline__ void init(const CoarseCycle<T>& a, T* lds) {
        lower.init(a, lds);  // the top level's rows fill the registers: last
        top.init(a, lds);
    }
    __device__ __forceinline__ void take(const T* r) { top.restrict_from(r); }
    __device__ __forceinline__ const T* cycle(const CoarseCycle<T>& a, T* lds) { return top.run(a, lds, lower); }
};
// level 0: the free node (1,1,1), slot 13 of 27 per component
template <int NC, typename T, int K>
struct Levels<NC, T, K, 0> {
    double b[NC];
    __device__ __forceinline__ void init(const CoarseCycle<T>&, T*) {}
    __device__ __forceinline__ void take(const T* r) {
        if (threadIdx.x != 0) return;
        constexpr int f1 = lvl_n(1) + 1, Nf = lvl_nodes(1);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const T* f = r + c * Nf + 2 + f1 * (2 + f1 * 2);
            T half = T(0);
#pragma unroll
            for (int k = 1; k < 8; ++k) {
                const int off = (k & 1) + f1 * (((k >> 1) & 1) + f1 * (k >> 2));
                half += f[off] + f[-off];
            }
            b[c] = (double)(f[0] + T(0.5) * half);
        }
    }
    __device__ __forceinline__ const T* cycle(const CoarseCycle<T>& a, T* lds) {
        if (threadIdx.x == 0) {
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                double v = 0.0;
#pragma unroll
                for (int d = 0; d < NC; ++d) v = fma(a.ainv[c * NC + d], b[d], v);
                lds[c * 27 + 13] = T(v);
            }
        }
        __syncthreads();
        return lds;
    }
};

template <int NC, typename T, int K>
__global__ void __launch_bounds__(ct(NC, sizeof(T))) k_coarse_cycle(const CoarseCycle<T> a) {
    __shared__ T lds[lds_values(NC, sizeof(T), K)];
    constexpr int CT = ct(NC, sizeof(T));
    const int tid = threadIdx.x;
    Levels<NC, T, K, K> levels;
    levels.init(a, lds);
    // the iterate buffers' boundary slots stay 0
    for (int i = tid; i < x_offset(NC, K + 1); i += CT) lds[i] = T(0);
#pragma unroll
    for (int s = 0; s < lvl_slots(NC, sizeof(T), K); ++s)
        if (levels.top.has(s)) levels.top.b[s] = a.b[levels.top.addr[s]];
    __syncthreads();
    const T* u = levels.cycle(a, lds);
    for (int i = tid; i < NC * lvl_nodes(K); i += CT) a.x[i] = u[i];
}

template <int NC, typename T>
hipError_t launch_k(int K, const CoarseCycle<T>& a, hipStream_t st) {
    switch (K) {
        case 1: hipLaunchKernelGGL((k_coarse_cycle<NC, T, 1>), dim3(1), dim3(ct(NC, sizeof(T))), 0, st, a); break;
        case 2: hipLaunchKernelGGL((k_coarse_cycle<NC, T, 2>), dim3(1), dim3(ct(NC, sizeof(T))), 0, st, a); break;
        case 3:
            if constexpr (max_level(NC) >= 3) {
                hipLaunchKernelGGL((k_coarse_cycle<NC, T, 3>), dim3(1), dim3(ct(NC, sizeof(T))), 0, st, a);
                break;
            }
            return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

int coarse_cycle_max_level(int ncomp) { return max_level(ncomp); }

template <typename T>
hipError_t launch_coarse_cycle(int ncomp, int K, const CoarseCycle<T>& a, hipStream_t st) {
    if ((ncomp != 1 && ncomp != 3) || K < 1 || K > max_level(ncomp)) return hipErrorInvalidValue;
    if (a.pre < 0 || a.post < 0 || a.pre > kCyclePasses || a.post > kCyclePasses) return hipErrorInvalidValue;
    if (!a.ainv || !a.b || !a.x) return hipErrorInvalidValue;
    for (int l = 1; l <= K; ++l)
        if ((ncomp == 1 ? !a.wts[l] : !a.nu[l]) || !a.dinv[l]) return hipErrorInvalidValue;
    return ncomp == 1 ? launch_k<1, T>(K, a, st) : launch_k<3, T>(K, a, st);
}

template hipError_t launch_coarse_cycle<double>(int, int, const CoarseCycle<double>&, hipStream_t);
template hipError_t launch_coarse_cycle<float>(int, int, const CoarseCycle<float>&, hipStream_t);

}  // namespace agca
