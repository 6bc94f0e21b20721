// Two products with the matrix-free level operator in one pass over memory: the two
// smoothing passes before the coarse correction with the residual (the first pass from zero
// is elementwise), or the two passes after it.  As separate element-loop passes (k_apply.hip)
// these read the coefficient, the right-hand side and the inverse diagonal twice and move
// the first product's result through memory; those passes run at the memory rate, so the
// V-cycle's time is the bytes it moves.  Algorithmic bytes per fine node, vector FP64:
// 144 here (b, D^-1, nu, x, r) against 120 + 120 before the correction, 144 against
// 144 + 168 after it.
//
// Layout of the work: a workgroup of 512 threads owns a column of TX x TY lattice cells and
// marches up in z, one cell per thread and step.  In step z the threads evaluate
//   * the first product A on cell layer z (x staged in a three-layer LDS ring), and
//   * the second product B on cell layer z - 2 of the first one's result y (two LDS layers),
// exchange corner sums as in k_apply.hip (x neighbours by DPP, y neighbours through LDS,
// z in registers), and after the exchange finalise y at node layer z and the output at
// node layer z - 2.  Two barriers per step: corner sums written -> read, y written -> read.
// The tile loses one row and column of cells per side and product: (TX-3) x (TY-3) nodes are
// written per layer.  A chunk of zc output layers takes zc + 4 steps.
//
// Why this shape: 32-wide rows (a wavefront covers two) and 16 rows are the largest tile
// whose vector FP64 state fits without spills: two products' carried sums, three coefficient
// layers and the loads in flight take 248 (before the correction) and 238 (after it) of the 256
// registers of 2 wavefronts per SIMD (one workgroup per compute unit, 137-157 KB of LDS); FP32 runs
// two workgroups per unit within 128 registers, of which the form with FP32 coefficients before the
// correction spills two (coarse levels; 21.3 us against 21.0 of the form after it at 65^3).  Node loads are issued one step ahead, in the order of their use (the
// wait counter is in order), right-hand side and inverse diagonal at the start of the step that
// ends with them: no register is copied from one that was just loaded, a copy would wait for
// every load in flight at the end of each step (vector FP64 V-cycle at 129^3 383 us with such
// copies, 360 without; 257^3 1970 and 1836; 513^3 BF16/FP32 7.55 and 7.32 ms).  Ordering the tiles in bands of
// rows so that the y halos are found in L2 measured slower (513^3 FP64 V-cycle, bands of
// 1 / 4 / 16 rows: 17.0 / 17.2 / 18.2 ms), as in k_apply.hip.
//
// Measured (MI355X, Chebyshev V(2,2), V-cycle before -> after): vector 513^3 FP64 23.2 ->
// 17.0 ms, FP32/BF16 11.5 -> 8.9 ms; 129^3 FP64 500 -> 416 us, FP32/BF16 269 -> 237 us;
// scalar 257^3 FP64 1.61 -> 1.04 ms.  Adding the coarse correction here instead of in a pass of
// its own (x read and written once more): vector 129^3 FP64 394 -> 384 us, FP32/BF16 237 -> 231,
// 513^3 15.3 -> 14.7 and 7.93 -> 7.84 ms, scalar 257^3 (k_scalar.hip) 803 -> 736 us.  At 513^3 the two FP64 passes take 6.2 and 5.6 ms and
// request 82 and 72 KB per workgroup and step, 5.0-5.2 TB/s: the streaming rate of a copy.  Counters
// (share of the time the vector ALUs issue / of a wavefront's cycles that wait for LDS): 513^3 BF16/FP32 90-98 % /
// 7.5 %, the issue limit; FP64 51-54 % / 5-9 %; 129^3 BF16/FP32 75-80 % / 7 %; FP64 44-46 % / 5-9 % at 2.9 TB/s, neither limit:
// two wavefronts per SIMD in steps with two barriers leave the rest idle.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <utility>

#include "cube_math.h"
#include "cube_tile.h"
#include "internal.h"

namespace agca {
namespace {

constexpr int TX = 32, TY = 16, NTH = TX * TY;
constexpr int OX = TX - 3, OY = TY - 3;  // nodes written per workgroup and layer
constexpr int TW = TX + 1;               // node row pitch of the staged layers
constexpr int TE = (TX + 1) * (TY + 1);  // nodes per staged layer

// wavefronts per SIMD the registers are allocated for
template <int NC, typename T>
struct Waves {
    static constexpr int value = NC == 3 && sizeof(T) == 8 ? 2 : 4;
};

// the six coefficients of a cell as loaded, decoded when used; a cell's are consecutive
static_assert(AGCA_ELEM_SOA == 0, "the two-product passes read a cell's six coefficients as one run");
template <typename NT>
struct CellNu;
template <>
struct CellNu<double> {
    u32x4 q[3];
    __device__ __forceinline__ void load(Rsrc r, uint32_t off) {
#pragma unroll
        for (int i = 0; i < 3; ++i) q[i] = __builtin_amdgcn_raw_buffer_load_b128(r, off + 16 * i, 0, 0);
    }
    __device__ __forceinline__ double get(int s) const {
        return __builtin_bit_cast(double, (s & 1) ? u32x2{q[s >> 1].z, q[s >> 1].w} : u32x2{q[s >> 1].x, q[s >> 1].y});
    }
};
template <>
struct CellNu<float> {
    u32x3 q[2];
    __device__ __forceinline__ void load(Rsrc r, uint32_t off) {
        q[0] = __builtin_amdgcn_raw_buffer_load_b96(r, off, 0, 0);
        q[1] = __builtin_amdgcn_raw_buffer_load_b96(r, off + 12, 0, 0);
    }
    __device__ __forceinline__ float get(int s) const { return __uint_as_float(q[s / 3][s % 3]); }
};
template <>
struct CellNu<uint16_t> {
    u32x3 q;
    __device__ __forceinline__ void load(Rsrc r, uint32_t off) { q = __builtin_amdgcn_raw_buffer_load_b96(r, off, 0, 0); }
    __device__ __forceinline__ float get(int s) const {
        return __uint_as_float((s & 1) ? (q[s >> 1] & 0xffff0000u) : (q[s >> 1] << 16));
    }
};

// The coefficients enter as stored; `scale` (LevelOp) multiplies the products: six multiplications of
// the coefficient per cell and product instead cost 129^3 FP32 / BF16 / FP64 V-cycles 221 -> 246,
// 218 -> 231 and 356 -> 361 us.  PRE: a1 is
// a1 + o1/om0 of the pass (a1 x1 + o1 D^-1 b with b = x1 / (om0 D^-1)), so the first pass
// needs no right-hand side.
template <int NC, typename T, typename NT, bool PRE>
__global__ void __launch_bounds__(NTH) __attribute__((amdgpu_waves_per_eu(Waves<NC, T>::value)))
k_smooth2(const int n, const int zc, const int gx, const int gy, const int gz, const T* __restrict__ x,
          const T* __restrict__ ec, const NT* __restrict__ nu, const T* __restrict__ b, const T* __restrict__ dinv,
          T* __restrict__ out, T* __restrict__ rout, const T scale, const T om0, const T a1, const T o1, const T a2, const T g2,
          const T o2) {
    __shared__ T xs[3][NC][TE + 64];       // staged x layers (64 slots absorb idle second stores)
    __shared__ T ys[2][NC][NTH + TX + 2];  // the first product's result, one value per thread
    __shared__ T fa[NC][2][NTH];           // corner sums passed up in y: first product
    __shared__ T fb[NC][2][NTH];           // second product
    // PRE: inverse diagonal of the own node, from its layer's load to its use two steps later
    __shared__ T ds[PRE ? 3 : 1][PRE ? NC : 1][PRE ? NTH : 1];
    using Coarse = CoarseTile<NC, T, TX, TY>;
    __shared__ typename Coarse::Tile es;  // POST: the coarse correction
    // POST: constants of a thread that are read back when used (in registers they spill, and the
    // reload from memory in every step waited for the loads in flight)
    __shared__ u32x4 lc[PRE ? 1 : NTH];
    const int cols = gx * gy;
    const int lin = tile_lin(cols, gz);
    const int bz = lin / cols, bc = lin - bz * cols;
    const int X0 = (bc % gx) * OX, Y0 = (bc / gx) * OY, Z0 = bz * zc;
    const int zend = min(Z0 + zc - 1, n);
    const int tid = threadIdx.x, tx = tid & (TX - 1), ty = tid / TX;
    const int cx = X0 - 2 + tx, cy = Y0 - 2 + ty;
    const int n1 = n + 1;
    const int64_t layer = (int64_t)n1 * n1, N = layer * n1, clayer = (int64_t)n * n;
    const uint32_t lbytes = (uint32_t)(layer * sizeof(T)), cbytes = (uint32_t)(clayer * 6 * sizeof(NT));
    // own node (the cell's lowest corner) and, for the first lanes, one node of the
    // tile's last column or last row
    auto node_off = [&](int X, int Y) {
        return X > 0 && X < n && Y > 0 && Y < n ? (uint32_t)(X + n1 * Y) * (uint32_t)sizeof(T) : kOut;
    };
    const uint32_t at = node_off(cx, cy);
    const bool has_b = tid < TX + TY + 1;
    const int ex = tid <= TY ? TX : tid - TY - 1, ey = tid <= TY ? tid : TY;
    const uint32_t at_b = has_b ? node_off(X0 - 2 + ex, Y0 - 2 + ey) : kOut;
    const int sa = ty * TW + tx;
    const int sb = has_b ? ey * TW + ex : TE + (tid & 63);
    const uint32_t cat = cx >= 0 && cx < n && cy >= 0 && cy < n ? (uint32_t)(cx + n * cy) * (uint32_t)(6 * sizeof(NT)) : kOut;
    const bool writer = tx >= 2 && tx <= TX - 2 && ty >= 2 && ty <= TY - 2 && cx <= n && cy <= n;
    const uint32_t at_w = writer ? (uint32_t)(cx + n1 * cy) * (uint32_t)sizeof(T) : kOut;
    // right-hand side of the second product's nodes, and (POST) of the first product's
    const uint32_t at_r = (PRE ? writer : tx >= 1 && ty >= 1) ? at : kOut;
    const int up = max(tid - TX, 0);

    // one node of a staged layer; PRE stages x1 = om0 D^-1 b.  Zero from the lattice boundary
    // on, and past the layers the chunk needs.
    struct Node {
        T v[NC], d[NC];
    };
    auto load_node = [&](int z, uint32_t off_xy, Node& t) {
        const bool zin = z > 0 && z < n && z <= zend + 2;
        const int64_t off = (int64_t)z * layer;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            t.v[c] = bload<T>(layer_of((PRE ? b : x) + off + c * N, zin, lbytes), off_xy);
            if constexpr (PRE) t.d[c] = bload<T>(layer_of(dinv + off + c * N, zin, lbytes), off_xy);
        }
    };
    Coarse coarse;
    if constexpr (!PRE) {
        coarse.init(ec, n, X0 - 2, Y0 - 2);
        lc[tid] = u32x4{at_b, (uint32_t)sb, coarse.slots(cx, cy, has_b ? X0 - 2 + ex : cx, has_b ? Y0 - 2 + ey : cy), coarse.offset()};
    }
    auto ext_offset = [&] { return PRE ? at_b : lc[PRE ? 0 : tid].x; };
    auto ext_slot = [&] { return PRE ? sb : (int)lc[PRE ? 0 : tid].y; };
    // layer z of the staged vector: the thread's node k into `slot`
    auto stage = [&](int z, int slot, const Node& t, int k) {
        T pe[NC];
        if constexpr (!PRE) Coarse::value(es, z, k, lc[tid].z, pe);
#pragma unroll
        for (int c = 0; c < NC; ++c) xs[(z + 6) % 3][c][slot] = PRE ? om0 * t.d[c] * t.v[c] : t.v[c] + pe[c];
    };
    auto load_nu = [&](int z, CellNu<NT>& r) {
        r.load(layer_of(nu + (int64_t)z * clayer * 6, z >= 0 && z < n && z <= zend + 1, cbytes), cat);
    };
    // contributions of one cell layer: sums over the x neighbours, [dy][dz]
    auto cell = [&](const T (&U)[8][NC], const CellNu<NT>& r, T (&P)[2][2][NC]) {
        T w[6];
#pragma unroll
        for (int s = 0; s < 6; ++s) w[s] = r.get(s);
        T F[8][NC];
        cell_flux<NC, T>(U, w, F);
#pragma unroll
        for (int dy = 0; dy < 2; ++dy)
#pragma unroll
            for (int dz = 0; dz < 2; ++dz)
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    P[dy][dz][c] = F[2 * dy + 4 * dz][c] + shr1_row(F[1 + 2 * dy + 4 * dz][c]);
    };
    auto bidx = [](int l) { return (l + 6) % 3; };

    // POST: the terms of the second pass known after the first, layers z-2 and z-1:
    // out = ch - oh (A y), ch = a2 y + g2 x + o2 D^-1 b
    T ch[2][NC], oh[2][NC];
    Node t[2], e[2];  // node layers Z0-2 and Z0-1
#pragma unroll
    for (int l = 0; l < 2; ++l) {
        load_node(Z0 - 2 + l, at, t[l]);
        load_node(Z0 - 2 + l, ext_offset(), e[l]);
    }
    T ev[NC];  // POST: the coarse layer to be stored next
    if constexpr (!PRE) {
        // these layers need coarse layers m0 and m0+1, the loop's first also m0+2 (Z0 odd) or
        // its next one (Z0 even)
        const int m0 = (Z0 - 2) >> 1;
        T v0[NC], v1[NC];
        coarse.load(m0, lc[tid].w, true, v0);
        coarse.load(m0 + 1, lc[tid].w, true, v1);
        coarse.load(m0 + 2, lc[tid].w, true, ev);
        coarse.store(es, m0, v0);
        coarse.store(es, m0 + 1, v1);
        __syncthreads();
    }
#pragma unroll
    for (int l = 0; l < 2; ++l) {
        stage(Z0 - 2 + l, sa, t[l], 0);
        stage(Z0 - 2 + l, ext_slot(), e[l], 1);
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if constexpr (PRE) ds[bidx(Z0 - 2 + l)][c][tid] = t[l].d[c];
    }
    CellNu<NT> r0, r1, r2, r3;  // layers z-2, z-1, z, z+1
    load_nu(Z0 - 2, r2);
    r0 = r2; r1 = r2;
    T ca[NC], cb[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        ca[c] = cb[c] = T(0);
        ch[0][c] = ch[1][c] = oh[0][c] = oh[1][c] = T(0);
    }
    Node own, ext;  // node layer z+2
    load_node(Z0, ext_offset(), ext);
    load_node(Z0, at, own);
    T bq[NC], dq[NC];  // POST: right-hand side and inverse diagonal of layer z; PRE: right-hand side of z-2
    auto load_rhs = [&](int z, T (&bv)[NC], T (&dv)[NC]) {
        const int zq = PRE ? z - 2 : z;
        const bool zin = zq > 0 && zq < n && zq >= Z0 - 1 && zq <= zend + 1;
        const int64_t off = (int64_t)zq * layer;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            bv[c] = bload<T>(layer_of(b + off + c * N, zin, lbytes), at_r);
            if constexpr (!PRE) dv[c] = bload<T>(layer_of(dinv + off + c * N, zin, lbytes), at_r);
        }
    };
    if constexpr (!PRE)
        if (Z0 & 1) {
            __syncthreads();
            coarse.store(es, (Z0 + 1) >> 1, ev);
        }
    __syncthreads();

    for (int z = Z0 - 2; z <= zend + 2; ++z) {
        load_rhs(z, bq, dq);
        // second product: cell layer z-2 of the first pass's result
        T PB[2][2][NC];
        {
            T U[8][NC];
            const int lo = z & 1, hi = lo ^ 1;  // layers z-2 and z-1
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    U[k][c] = ys[lo][c][tid + (k >> 1) * TX + (k & 1)];
                    U[k + 4][c] = ys[hi][c][tid + (k >> 1) * TX + (k & 1)];
                }
            cell(U, r0, PB);
        }
        if constexpr (!PRE)
            if (!(z & 1)) coarse.store(es, (z >> 1) + 2, ev);
        stage(z + 2, ext_slot(), ext, 1);
        __builtin_amdgcn_sched_barrier(0);
        load_nu(z + 1, r3);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            fb[c][0][tid] = PB[1][0][c];
            fb[c][1][tid] = PB[1][1][c];
            cb[c] += PB[0][0][c];
        }
        __builtin_amdgcn_sched_barrier(0);
        // first product: cell layer z
        T PA[2][2][NC];
        {
            T U[8][NC];
            const int lo = bidx(z), hi = bidx(z + 1);
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    U[k][c] = xs[lo][c][sa + (k >> 1) * TW + (k & 1)];
                    U[k + 4][c] = xs[hi][c][sa + (k >> 1) * TW + (k & 1)];
                }
            cell(U, r2, PA);
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            fa[c][0][tid] = PA[1][0][c];
            fa[c][1][tid] = PA[1][1][c];
        }
        stage(z + 2, sa, own, 0);
        if constexpr (PRE) {
#pragma unroll
            for (int c = 0; c < NC; ++c) ds[bidx(z + 2)][c][tid] = own.d[c];
        }
        if constexpr (!PRE) coarse.load((z + 5) >> 1, lc[tid].w, z & 1, ev);
        load_node(z + 3, ext_offset(), ext);
        load_node(z + 3, at, own);
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        // boundary nodes have self = dinv = b = 0, hence y = 0
        const bool wA = z >= Z0 && z <= zend, wB = z - 2 >= Z0 && z - 2 <= zend;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const T av = ca[c] + (PA[0][0][c] + fa[c][0][up]);
            ca[c] = PA[0][1][c] + fa[c][1][up];
            const T bv = cb[c] + fb[c][0][up];
            cb[c] = PB[0][1][c] + fb[c][1][up];
            const T self = xs[bidx(z)][c][sa];
            const Rsrc wr = layer_of((PRE ? rout : out) + (int64_t)(z - 2) * layer + c * N, wB, lbytes);
            T y;
            if constexpr (PRE) {
                y = a1 * self - o1 * ds[bidx(z)][c][tid] * (scale * av);
                bstore<T>(layer_of(out + (int64_t)z * layer + c * N, wA, lbytes), at_w, y);
                bstore<T>(wr, at_w, at != kOut && z > 2 && z - 2 < n ? fma(-scale, bv, bq[c]) : T(0));
            } else {
                y = a1 * self + o1 * dq[c] * fma(-scale, av, bq[c]);
                bstore<T>(wr, at_w, ch[0][c] - oh[0][c] * bv);
                ch[0][c] = ch[1][c];
                oh[0][c] = oh[1][c];
                const T od = o2 * dq[c];
                oh[1][c] = scale * od;
                ch[1][c] = a2 * y + g2 * self + od * bq[c];
            }
            ys[z & 1][c][tid] = y;
        }
        r0 = r1; r1 = r2; r2 = r3;
        __syncthreads();
    }
}

template <int NC, typename T, typename NT, bool PRE>
hipError_t launch_t(const LevelOp<T>& op, const Smooth2<T>& a, hipStream_t st) {
    const int n = op.n;
    static const std::pair<int, int> fit = workgroups_fit(k_smooth2<NC, T, NT, PRE>, NTH);
    const int gx = (n + OX) / OX, gy = (n + OY) / OY;
    const int gz = pick_chunks(n, (int64_t)gx * gy, fit.first, fit.second);
    const int zc = (n + gz) / gz;
    hipLaunchKernelGGL((k_smooth2<NC, T, NT, PRE>), dim3((unsigned)(gx * gy * gz)), dim3(NTH), 0, st, n, zc, gx, gy, gz, a.x, a.e, reinterpret_cast<const NT*>(op.nu), a.b, op.dinv, a.out, a.r, T(op.scale), a.om0,
                       PRE ? a.first() : a.a1, a.o1, a.a2, a.g2, a.o2);
    return hipGetLastError();
}

template <int NC, typename T, bool PRE>
hipError_t launch_nu(const LevelOp<T>& op, const Smooth2<T>& a, hipStream_t st) {
    if constexpr (sizeof(T) == 8) {
        return op.nu_kind == AGCA_F64 ? launch_t<NC, T, double, PRE>(op, a, st) : hipErrorInvalidValue;
    } else {
        if (op.nu_kind == AGCA_F32) return launch_t<NC, T, float, PRE>(op, a, st);
        return op.nu_kind == AGCA_BF16 ? launch_t<NC, T, uint16_t, PRE>(op, a, st) : hipErrorInvalidValue;
    }
}

}  // namespace

template <typename T>
hipError_t launch_smooth2(int ncomp, bool pre, const LevelOp<T>& op, const Smooth2<T>& a, hipStream_t st) {
    if (!op.nu || !op.dinv || op.n < 2 || !a.b || !a.out || (pre ? !a.r : !a.x || !a.e || a.x == a.out))
        return hipErrorInvalidValue;
    if (ncomp == 1) return pre ? launch_nu<1, T, true>(op, a, st) : launch_nu<1, T, false>(op, a, st);
    return pre ? launch_nu<3, T, true>(op, a, st) : launch_nu<3, T, false>(op, a, st);
}

template hipError_t launch_smooth2<double>(int, bool, const LevelOp<double>&, const Smooth2<double>&, hipStream_t);
template hipError_t launch_smooth2<float>(int, bool, const LevelOp<float>&, const Smooth2<float>&, hipStream_t);

}  // namespace agca
