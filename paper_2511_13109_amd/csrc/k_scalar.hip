// Scalar operators (-div nu grad u) in their seven-point form.
//
// Every path step of a Kuhn simplex is a lattice edge along an axis, and the scalar element
// matrix is the path Laplacian (eq. (2.3), kuhn.h), so the assembled operator couples a node
// with its six axis neighbours only:
//   (A u)(p) = sum over the six edges (p, q) of W(p, q) (u(p) - u(q)),
// W the sum of nu_e h/6 over the simplices that have the edge as a path step (up to 8 in the
// four cells around it).  Three weights per node (the edges to x+1, y+1, z+1) replace the six
// coefficients per cell of the element loop: 24 against 48 bytes per node in FP64, 12 against
// 24 in FP32, a seven-point gather instead of 8 corners, and the same operator up to the
// order of the additions.  The weights are formed in FP64 once per coefficient, from the
// coefficient the operator uses (rounded to BF16 where the V-cycle's finest one is).
//
// Measured against the element loop: product 257^3 FP64 249 -> 159 us (680 MB: 4.3 TB/s), 513^3
// 1945 -> 1203 us; V-cycle (Chebyshev 2, 2; before with one element-loop product per pass) 129^3
// FP64 222 -> 118 us, 257^3 1627 -> 680, 513^3 FP64 12137 -> 5390, FP32 6536 -> 2750.
//
// Layout: W[a * N + p], a = 0, 1, 2 the edge from node p along axis a, N = (n+1)^3; 0 where
// the edge leaves the lattice.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <utility>

#include "cube_math.h"
#include "cube_tile.h"
#include "internal.h"

namespace agca {
namespace {

constexpr int NT = 256;

// whether simplex s steps along axis a from cell corner m
AGCA_HDC constexpr bool steps_from(int s, int a, int m) {
    return (axis1(s) == a && path_corner(s, 0) == m) || (axis2(s) == a && path_corner(s, 1) == m) ||
           (axis3(s) == a && path_corner(s, 2) == m);
}

__device__ __forceinline__ double nu_value(double v) { return v; }
__device__ __forceinline__ double nu_value(uint16_t v) { return (double)bf16_to_float(v); }

template <typename NT_, typename T>
__global__ void __launch_bounds__(NT)
k_weights(int n, const NT_* __restrict__ nu, double scale, T* __restrict__ W, float* __restrict__ W32) {
    const int64_t n1 = n + 1, N = n1 * n1 * n1, cells = (int64_t)n * n * n;
    const int64_t p = blockIdx.x * (int64_t)NT + threadIdx.x;
    if (p >= N) return;
    int q[3];
    node_coords(p, n, q[0], q[1], q[2]);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int b = (a + 1) % 3, c = (a + 2) % 3;
        double w = 0.0;
        if (q[a] < n) {
#pragma unroll
            for (int o = 0; o < 4; ++o) {
                // the cell that has the edge's lower node as its corner m
                const int m = ((o & 1) << b) | ((o >> 1) << c);
                const int cx = q[0] - (m & 1), cy = q[1] - ((m >> 1) & 1), cz = q[2] - (m >> 2);
                if (cx < 0 || cy < 0 || cz < 0 || cx >= n || cy >= n || cz >= n) continue;
                const int64_t cell = cx + (int64_t)n * (cy + (int64_t)n * cz);
#pragma unroll
                for (int s = 0; s < 6; ++s)
                    if (steps_from(s, a, m)) w += nu_value(nu[elem_slot(s, cell, cells)]);
            }
        }
        W[a * N + p] = T(w * scale);
        if (W32) W32[a * N + p] = float(w * scale);
    }
}

// the value a pass writes, from A u, u, and the node's right-hand side, inverse diagonal and
// previous iterate (Sweep, internal.h)
template <int MODE, typename T>
__device__ __forceinline__ T pass_value(T av, T u, T b, T d, T xp, T omega, T alpha, T gamma) {
    if constexpr (MODE == MODE_APPLY || MODE == MODE_APPLY_DOT) return av;
    else if constexpr (MODE == MODE_RESIDUAL) return b - av;
    else if constexpr (MODE == MODE_CHEB) return fma(omega * d, b - av, fma(gamma, xp, alpha * u));
    else return fma(omega * d, b - av, alpha * u);
}

__device__ __forceinline__ void store_partial(double v, double* __restrict__ out) {
    __shared__ double red[NT / 64];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < NT / 64; ++w) s += red[w];
        *out = s;
    }
}

// One product on a small level, one thread per node: every load of a node in flight at once,
// no march.  Bound by latency.  out may be b or xprev (a residual in place, a Chebyshev pass into
// the previous iterate's buffer): a node's values are read before its result is written.
template <typename T, int MODE>
__global__ void __launch_bounds__(NT)
k_node7(int n, const T* __restrict__ W, const T* __restrict__ u, const T* b,
        const T* __restrict__ dinv, T* out, T omega, T alpha, T gamma, const T* xprev,
        double* __restrict__ partial) {
    const int n1 = n + 1;
    const uint32_t N = (uint32_t)n1 * n1 * n1, p = blockIdx.x * NT + threadIdx.x;
    double dot = 0.0;
    if (p < N) {
        int x, y, z;
        node_coords(p, n, x, y, z);
        T v = T(0);
        if (x > 0 && y > 0 && z > 0 && x < n && y < n && z < n) {
            const uint32_t sy = n1, sz = n1 * n1;
            const T uc = u[p];
            // boundary values count 0
            const T xm = u[p - 1], xq = u[p + 1], ym = u[p - sy], yq = u[p + sy], zm = u[p - sz], zq = u[p + sz];
            const T wx = W[p], wxm = W[p - 1], wy = W[N + p], wym = W[N + p - sy], wz = W[2 * N + p], wzm = W[2 * N + p - sz];
            T av = wxm * (uc - (x > 1 ? xm : T(0)));
            av = fma(wx, uc - (x < n - 1 ? xq : T(0)), av);
            av = fma(wym, uc - (y > 1 ? ym : T(0)), av);
            av = fma(wy, uc - (y < n - 1 ? yq : T(0)), av);
            av = fma(wzm, uc - (z > 1 ? zm : T(0)), av);
            av = fma(wz, uc - (z < n - 1 ? zq : T(0)), av);
            constexpr bool SMOOTH = MODE == MODE_JACOBI || MODE == MODE_CHEB;
            v = pass_value<MODE>(av, uc, MODE == MODE_RESIDUAL || SMOOTH ? b[p] : T(0), SMOOTH ? dinv[p] : T(0),
                                 MODE == MODE_CHEB ? xprev[p] : T(0), omega, alpha, gamma);
            if (MODE == MODE_APPLY_DOT) dot = (double)uc * (double)av;
        }
        out[p] = v;
    }
    if (MODE == MODE_APPLY_DOT) store_partial(dot, partial + blockIdx.x);
}

// One product on a large level.  A wavefront owns 64 nodes of a lattice row and marches a
// chunk of z layers, no LDS and no barriers: x neighbours by DPP (the row's two outer ones by
// a load that only the end lanes take part in), y neighbours from cache, the z flux carried in
// a register, every load issued one step ahead.  Interior nodes number 2^k - 1 per row, so
// 64-wide rows leave no lanes idle.  Bound by memory: 40 bytes per node (FP64 apply).  out may be b
// or xprev, as in k_node7.
template <typename T, int MODE>
__global__ void __launch_bounds__(NT)
k_march7(const int n, const int zc, const int gx, const int gy, const int gz, const T* __restrict__ W,
         const T* __restrict__ u, const T* b, const T* __restrict__ dinv, T* out,
         const T omega, const T alpha, const T gamma, const T* xprev, double* __restrict__ partial) {
    const int cols = gx * gy, lin = tile_lin(cols, gz), bz = lin / cols, bc = lin - bz * cols;
    const int lane = threadIdx.x & 63;
    const int x = 1 + 64 * (bc % gx) + lane;
    const int y = __builtin_amdgcn_readfirstlane((bc / gx) * (NT / 64) + (int)(threadIdx.x >> 6));
    const int Z0 = bz * zc, zend = min(Z0 + zc - 1, n);
    const int n1 = n + 1;
    const int64_t layer = (int64_t)n1 * n1, N = layer * n1;
    const uint32_t lbytes = (uint32_t)(layer * sizeof(T)), row = (uint32_t)(n1 * sizeof(T));
    const bool in = x < n && y > 0 && y < n;
    const uint32_t at = in ? (uint32_t)(x + n1 * y) * (uint32_t)sizeof(T) : kOut;
    const uint32_t at_yq = in && y < n - 1 ? at + row : kOut, at_ym = in && y > 1 ? at - row : kOut;
    const uint32_t at_wm = in ? at - row : kOut;
    // the neighbours beyond the wavefront's ends
    const uint32_t at_e = !in ? kOut : lane == 0 && x > 1 ? at - (uint32_t)sizeof(T)
                        : lane == 63 && x < n - 1 ? at + (uint32_t)sizeof(T) : kOut;
    const uint32_t at_we = in && lane == 0 ? at - (uint32_t)sizeof(T) : kOut;
    // stores: interior nodes and, by the lanes next to them, the row's two boundary nodes
    const bool row_ok = y <= n;
    const uint32_t at_w = row_ok && x < n ? (uint32_t)(x + n1 * y) * (uint32_t)sizeof(T) : kOut;
    const uint32_t at_wb = !row_ok ? kOut : x == 1 ? (uint32_t)(n1 * y) * (uint32_t)sizeof(T)
                         : x == n ? (uint32_t)(n + n1 * y) * (uint32_t)sizeof(T) : kOut;
    constexpr bool SMOOTH = MODE == MODE_JACOBI || MODE == MODE_CHEB;
    constexpr bool NEEDS_B = MODE == MODE_RESIDUAL || SMOOTH;
    struct Step {  // what the nodes of one layer need beside u(z) and u(z+1)
        T yq, ym, e, wx, wy, wym, wz, we, b, d, xp;
    };
    auto load = [&](int z, Step& s) {
        const bool zin = z > 0 && z < n && z <= zend;
        const int64_t off = (int64_t)z * layer;
        const Rsrc ru = layer_of(u + off, zin, lbytes), rx = layer_of(W + off, zin, lbytes),
                   ry = layer_of(W + N + off, zin, lbytes);
        s.yq = bload<T>(ru, at_yq);
        s.ym = bload<T>(ru, at_ym);
        s.e = bload<T>(ru, at_e);
        s.wx = bload<T>(rx, at);
        s.we = bload<T>(rx, at_we);
        s.wy = bload<T>(ry, at);
        s.wym = bload<T>(ry, at_wm);
        s.wz = bload<T>(layer_of(W + 2 * N + off, z >= 0 && z < n && z <= zend, lbytes), at);
        if constexpr (NEEDS_B) s.b = bload<T>(layer_of(b + off, zin, lbytes), at);
        if constexpr (SMOOTH) s.d = bload<T>(layer_of(dinv + off, zin, lbytes), at);
        if constexpr (MODE == MODE_CHEB) s.xp = bload<T>(layer_of(xprev + off, zin, lbytes), at);
    };
    auto load_u = [&](int z) {
        return bload<T>(layer_of(u + (int64_t)z * layer, z > 0 && z < n && z <= zend + 1, lbytes), at);
    };
    double dot = 0.0;
    const T wz0 = bload<T>(layer_of(W + 2 * N + (int64_t)(Z0 - 1) * layer, Z0 > 0, lbytes), at);
    const T um = load_u(Z0 - 1);
    const T uc = load_u(Z0), uq = load_u(Z0 + 1);
    T fz = wz0 * (uc - um);  // flux from layer z-1 into z
    // layer z, its values in cur and u(z), u(z+1) in uc, uq; loads layer z+1's into nxt, u(z+2) into un
    auto step = [&](int z, const Step& cur, Step& nxt, const T uc, const T uq, T& un) {
        load(z + 1, nxt);
        un = load_u(z + 2);
        // (every lane takes part in the exchanges; the ends then replace what they got)
        const T right = shl1_row(uc);
        const T fx = cur.wx * ((lane == 63 ? cur.e : right) - uc);
        const T left = shr1_row(fx);
        const T fxm = lane == 0 ? cur.we * (uc - cur.e) : left;
        const T fy = cur.wy * (cur.yq - uc), fym = cur.wym * (uc - cur.ym);
        const T fq = cur.wz * (uq - uc);
        // layer 0 and n: no loads, uc = 0, but fz may not vanish: boundary nodes are 0
        const T av = z > 0 && z < n ? ((fxm - fx) + (fym - fy)) + (fz - fq) : T(0);
        fz = fq;
        const T v = pass_value<MODE>(av, uc, cur.b, cur.d, cur.xp, omega, alpha, gamma);
        if (MODE == MODE_APPLY_DOT) dot += (double)uc * (double)av;
        const Rsrc ro = layer_of(out + (int64_t)z * layer, true, lbytes);
        bstore<T>(ro, at_w, in ? v : T(0));
        bstore<T>(ro, at_wb, T(0));
    };
    // registers in turn: a copy from those just loaded would wait for the loads
    Step s0, s1;
    T u0 = uc, u1 = uq, u2;
    load(Z0, s0);
    for (int z = Z0;;) {
        step(z, s0, s1, u0, u1, u2);
        if (++z > zend) break;
        step(z, s1, s0, u1, u2, u0);
        if (++z > zend) break;
        step(z, s0, s1, u2, u0, u1);
        if (++z > zend) break;
        step(z, s1, s0, u0, u1, u2);
        if (++z > zend) break;
        step(z, s0, s1, u1, u2, u0);
        if (++z > zend) break;
        step(z, s1, s0, u2, u0, u1);
        if (++z > zend) break;
    }
    if (MODE == MODE_APPLY_DOT) store_partial(dot, partial + blockIdx.x);
}

// rows of nodes, boundary included, per z chunk: gx x gy workgroups
struct March7Grid {
    int gx, gy, gz, zc;
};
// the marching kernel from here on.  At 128 cells it is the faster form (FP64 product 17.0 us, one
// thread per node 23.8); at 64 the slower one (5.1 and 3.9, smoothing pass 5.9 and 5.2), so the
// line could be higher; V-cycles run two products per pass there and do not notice (57.5 us with
// either).
constexpr int kMarchMinN = 64;
March7Grid march7_grid(int n) {
    March7Grid g;
    g.gx = (n + 63) / 64;  // x = 1 .. n: the lane past the interior writes the boundary node n
    g.gy = (n + 1 + NT / 64 - 1) / (NT / 64);
    // chunks of 32 layers (each starts with two more loads of u and one of W), shorter while
    // fewer than 2048 workgroups (8 per compute unit) would run; chunks of 16 to 64 layers and 2
    // to 16 rows per workgroup measure alike (257^3 FP64 163-173 us)
    int zc = 32;
    while (zc > 4 && (int64_t)g.gx * g.gy * ((n + zc) / zc) < 2048) zc /= 2;
    g.gz = (n + zc) / zc;
    g.zc = (n + g.gz) / g.gz;
    return g;
}

template <typename T, int MODE>
hipError_t launch_one(int n, const T* W, const T* u, const T* b, const T* dinv, T* out, const Sweep<T>& sw,
                      hipStream_t st, double* partial = nullptr, int* nblocks = nullptr) {
    if (n < kMarchMinN) {
        const int64_t N = (int64_t)(n + 1) * (n + 1) * (n + 1);
        const int g = (int)((N + NT - 1) / NT);
        if (nblocks) *nblocks = g;
        hipLaunchKernelGGL((k_node7<T, MODE>), dim3((unsigned)g), dim3(NT), 0, st, n, W, u, b, dinv, out, sw.omega,
                           sw.alpha, sw.gamma, sw.xprev, partial);
    } else {
        const March7Grid g = march7_grid(n);
        const int nwg = g.gx * g.gy * g.gz;
        if (nblocks) *nblocks = nwg;
        hipLaunchKernelGGL((k_march7<T, MODE>), dim3((unsigned)nwg), dim3(NT), 0, st, n, g.zc, g.gx, g.gy, g.gz, W, u, b,
                           dinv, out, sw.omega, sw.alpha, sw.gamma, sw.xprev, partial);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Two products in one pass: k_smooth2.hip's scheme with the seven-point form (same tile,
// same steps; the thread of a cell is the thread of its lowest node).
// ---------------------------------------------------------------------------
constexpr int TX = 32, TY = 16, NTH = TX * TY;
constexpr int OX = TX - 3, OY = TY - 3;
constexpr int TW = TX + 1, TE = (TX + 1) * (TY + 1);

template <typename T, bool PRE>
__global__ void __launch_bounds__(NTH)
k_two7(const int n, const int zc, const int gx, const int gy, const int gz, const T* __restrict__ x,
       const T* __restrict__ ec, const T* __restrict__ W, const T* __restrict__ b, const T* __restrict__ dinv,
       T* __restrict__ out, T* __restrict__ rout, const T om0, const T a1, const T o1, const T a2, const T g2,
       const T o2) {
    using Coarse = CoarseTile<1, T, TX, TY>;
    __shared__ typename Coarse::Tile es;  // POST: the coarse correction
    __shared__ T xs[3][TE + 64];
    __shared__ T ys[2][NTH + TX + 2];
    __shared__ T fa[NTH], fb[NTH];
    __shared__ T ds[PRE ? 3 : 1][PRE ? NTH : 1];
    const int cols = gx * gy;
    const int lin = tile_lin(cols, gz);
    const int bz = lin / cols, bc = lin - bz * cols;
    const int X0 = (bc % gx) * OX, Y0 = (bc / gx) * OY, Z0 = bz * zc;
    const int zend = min(Z0 + zc - 1, n);
    const int tid = threadIdx.x, tx = tid & (TX - 1), ty = tid / TX;
    const int cx = X0 - 2 + tx, cy = Y0 - 2 + ty;
    const int n1 = n + 1;
    const int64_t layer = (int64_t)n1 * n1, N = layer * n1;
    const uint32_t lbytes = (uint32_t)(layer * sizeof(T));
    auto node_off = [&](int X, int Y) {
        return X > 0 && X < n && Y > 0 && Y < n ? (uint32_t)(X + n1 * Y) * (uint32_t)sizeof(T) : kOut;
    };
    const uint32_t at = node_off(cx, cy);
    const bool has_b = tid < TX + TY + 1;
    const int ex = tid <= TY ? TX : tid - TY - 1, ey = tid <= TY ? tid : TY;
    const uint32_t at_b = has_b ? node_off(X0 - 2 + ex, Y0 - 2 + ey) : kOut;
    const int sa = ty * TW + tx;
    const int sb = has_b ? ey * TW + ex : TE + (tid & 63);
    // weights: every lattice node (an edge may start on the boundary)
    const uint32_t wat = cx >= 0 && cx <= n && cy >= 0 && cy <= n ? (uint32_t)(cx + n1 * cy) * (uint32_t)sizeof(T) : kOut;
    const bool writer = tx >= 2 && tx <= TX - 2 && ty >= 2 && ty <= TY - 2 && cx <= n && cy <= n;
    const uint32_t at_w = writer ? wat : kOut;
    const uint32_t at_r = (PRE ? writer : tx >= 1 && ty >= 1) ? at : kOut;
    const int up = max(tid - TX, 0);
    struct Node {
        T v, d;
    };
    auto load_node = [&](int z, uint32_t off_xy, Node& t) {
        const bool zin = z > 0 && z < n && z <= zend + 2;
        t.v = bload<T>(layer_of((PRE ? b : x) + (int64_t)z * layer, zin, lbytes), off_xy);
        if constexpr (PRE) t.d = bload<T>(layer_of(dinv + (int64_t)z * layer, zin, lbytes), off_xy);
    };
    Coarse coarse;
    uint32_t slots = 0, at_e = 0;
    if constexpr (!PRE) {
        coarse.init(ec, n, X0 - 2, Y0 - 2);
        slots = coarse.slots(cx, cy, has_b ? X0 - 2 + ex : cx, has_b ? Y0 - 2 + ey : cy);
        at_e = coarse.offset();
    }
    // layer z of the staged vector: the thread's node k into `slot`
    auto stage = [&](int z, int slot, const Node& t, int k) {
        T pe[1];
        if constexpr (!PRE) Coarse::value(es, z, k, slots, pe);
        xs[(z + 6) % 3][slot] = PRE ? om0 * t.d * t.v : t.v + pe[0];
    };
    struct Edges {
        T w[3];
    };
    auto load_w = [&](int z, Edges& r) {
        const bool zin = z >= 0 && z <= n && z <= zend + 1;
#pragma unroll
        for (int a = 0; a < 3; ++a) r.w[a] = bload<T>(layer_of(W + a * N + (int64_t)z * layer, zin, lbytes), wat);
    };
    // node sums without the y neighbour's flux: own, passed up in y, passed up in z
    auto node = [&](T c, T xq, T yq, T zq, const Edges& r, T& own, T& fy, T& fz) {
        const T fx = r.w[0] * (xq - c);
        fy = r.w[1] * (yq - c);
        fz = r.w[2] * (zq - c);
        own = ((shr1_row(fx) - fx) - fy) - fz;
    };
    auto bidx = [](int l) { return (l + 6) % 3; };
    T ch[2] = {T(0), T(0)}, oh[2] = {T(0), T(0)};
    Node t[2], e[2];  // node layers Z0-2 and Z0-1
#pragma unroll
    for (int l = 0; l < 2; ++l) {
        load_node(Z0 - 2 + l, at, t[l]);
        load_node(Z0 - 2 + l, at_b, e[l]);
    }
    T ev[1];  // POST: the coarse layer to be stored next
    if constexpr (!PRE) {
        // these layers need coarse layers m0 and m0+1, the loop's first also m0+2 (Z0 odd) or
        // its next one (Z0 even)
        const int m0 = (Z0 - 2) >> 1;
        T v0[1], v1[1];
        coarse.load(m0, at_e, true, v0);
        coarse.load(m0 + 1, at_e, true, v1);
        coarse.load(m0 + 2, at_e, true, ev);
        coarse.store(es, m0, v0);
        coarse.store(es, m0 + 1, v1);
        __syncthreads();
    }
#pragma unroll
    for (int l = 0; l < 2; ++l) {
        stage(Z0 - 2 + l, sa, t[l], 0);
        stage(Z0 - 2 + l, sb, e[l], 1);
        if constexpr (PRE) ds[bidx(Z0 - 2 + l)][tid] = t[l].d;
    }
    Edges r0, r1, r2, r3;
    load_w(Z0 - 2, r2);
    r0 = r2; r1 = r2;
    T ca = T(0), cb = T(0);
    Node own, ext;
    load_node(Z0, at_b, ext);
    load_node(Z0, at, own);
    T bq, dq = T(0);
    auto load_rhs = [&](int z, T& bv, T& dv) {
        const int zq = PRE ? z - 2 : z;
        const bool zin = zq > 0 && zq < n && zq >= Z0 - 1 && zq <= zend + 1;
        bv = bload<T>(layer_of(b + (int64_t)zq * layer, zin, lbytes), at_r);
        if constexpr (!PRE) dv = bload<T>(layer_of(dinv + (int64_t)zq * layer, zin, lbytes), at_r);
    };
    if constexpr (!PRE)
        if (Z0 & 1) {
            __syncthreads();
            coarse.store(es, (Z0 + 1) >> 1, ev);
        }
    __syncthreads();
    for (int z = Z0 - 2; z <= zend + 2; ++z) {
        load_rhs(z, bq, dq);
        T ownB, fyB, fzB, ownA, fyA, fzA;
        {
            const int lo = z & 1, hi = lo ^ 1;  // layers z-2 and z-1
            node(ys[lo][tid], ys[lo][tid + 1], ys[lo][tid + TX], ys[hi][tid], r0, ownB, fyB, fzB);
        }
        if constexpr (!PRE)
            if (!(z & 1)) coarse.store(es, (z >> 1) + 2, ev);
        stage(z + 2, sb, ext, 1);
        load_w(z + 1, r3);
        fb[tid] = fyB;
        cb += ownB;
        const int lo = bidx(z), hi = bidx(z + 1);
        const T self = xs[lo][sa];
        node(self, xs[lo][sa + 1], xs[lo][sa + TW], xs[hi][sa], r2, ownA, fyA, fzA);
        fa[tid] = fyA;
        stage(z + 2, sa, own, 0);
        if constexpr (PRE) ds[bidx(z + 2)][tid] = own.d;
        if constexpr (!PRE) coarse.load((z + 5) >> 1, at_e, z & 1, ev);
        load_node(z + 3, at_b, ext);
        load_node(z + 3, at, own);
        __syncthreads();
        const bool wA = z >= Z0 && z <= zend, wB = z - 2 >= Z0 && z - 2 <= zend;
        const T av = ca + (ownA + fa[up]);
        ca = fzA;
        const T bv = cb + fb[up];
        cb = fzB;
        const Rsrc wr = layer_of((PRE ? rout : out) + (int64_t)(z - 2) * layer, wB, lbytes);
        T y;
        if constexpr (PRE) {
            y = a1 * self - o1 * ds[lo][tid] * av;
            bstore<T>(layer_of(out + (int64_t)z * layer, wA, lbytes), at_w, y);
            bstore<T>(wr, at_w, at != kOut && z > 2 && z - 2 < n ? bq - bv : T(0));
        } else {
            y = a1 * self + o1 * dq * (bq - av);
            bstore<T>(wr, at_w, ch[0] - oh[0] * bv);
            ch[0] = ch[1];
            oh[0] = oh[1];
            oh[1] = o2 * dq;
            ch[1] = a2 * y + g2 * self + oh[1] * bq;
        }
        ys[z & 1][tid] = y;
        r0 = r1; r1 = r2; r2 = r3;
        __syncthreads();
    }
}

template <typename T, bool PRE>
hipError_t launch_two(int n, const T* W, const T* dinv, const Smooth2<T>& a, hipStream_t st) {
    static const std::pair<int, int> fit = workgroups_fit(k_two7<T, PRE>, NTH);
    const int gx = (n + OX) / OX, gy = (n + OY) / OY;
    const int gz = pick_chunks(n, (int64_t)gx * gy, fit.first, fit.second);
    hipLaunchKernelGGL((k_two7<T, PRE>), dim3((unsigned)(gx * gy * gz)), dim3(NTH), 0, st, n, (n + gz) / gz, gx, gy, gz,
                       a.x, a.e, W, a.b, dinv, a.out, a.r, a.om0, PRE ? a.first() : a.a1, a.o1, a.a2, a.g2, a.o2);
    return hipGetLastError();
}

}  // namespace

template <typename T>
hipError_t launch_weights(int n, const double* nu, const uint16_t* nu_bf16, T* W, float* W32, hipStream_t st) {
    if ((!nu && !nu_bf16) || !W || n < 2) return hipErrorInvalidValue;
    const int64_t N = (int64_t)(n + 1) * (n + 1) * (n + 1);
    const dim3 g((unsigned)((N + NT - 1) / NT));
    if (nu_bf16)
        hipLaunchKernelGGL((k_weights<uint16_t, T>), g, dim3(NT), 0, st, n, nu_bf16, nu_scale(n, true), W, W32);
    else
        hipLaunchKernelGGL((k_weights<double, T>), g, dim3(NT), 0, st, n, nu, nu_scale(n, false), W, W32);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_product7(int mode, int n, const T* W, const T* u, const T* b, const T* dinv, T* out,
                           const Sweep<T>& sw, hipStream_t st) {
    if (!W || !u || !out || n < 2 || (mode != MODE_APPLY && !b)) return hipErrorInvalidValue;
    if ((mode == MODE_JACOBI || mode == MODE_CHEB) && !dinv) return hipErrorInvalidValue;
    if (mode == MODE_CHEB && !sw.xprev) return hipErrorInvalidValue;
    switch (mode) {
        case MODE_APPLY: return launch_one<T, MODE_APPLY>(n, W, u, b, dinv, out, sw, st);
        case MODE_RESIDUAL: return launch_one<T, MODE_RESIDUAL>(n, W, u, b, dinv, out, sw, st);
        case MODE_JACOBI: return launch_one<T, MODE_JACOBI>(n, W, u, b, dinv, out, sw, st);
        case MODE_CHEB: return launch_one<T, MODE_CHEB>(n, W, u, b, dinv, out, sw, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_product7_dot(int n, const double* W, const double* u, double* out, double* partial, int* nblocks,
                               hipStream_t st) {
    if (!W || !u || !out || !partial || !nblocks || n < 2) return hipErrorInvalidValue;
    return launch_one<double, MODE_APPLY_DOT>(n, W, u, nullptr, nullptr, out, Sweep<double>{}, st, partial, nblocks);
}
int product7_blocks(int n) {
    if (n < kMarchMinN) return (int)(((int64_t)(n + 1) * (n + 1) * (n + 1) + NT - 1) / NT);
    const March7Grid g = march7_grid(n);
    return g.gx * g.gy * g.gz;
}

template <typename T>
hipError_t launch_two7(bool pre, int n, const T* W, const T* dinv, const Smooth2<T>& a, hipStream_t st) {
    if (!W || !dinv || n < 2 || !a.b || !a.out || (pre ? !a.r : !a.x || !a.e || a.x == a.out)) return hipErrorInvalidValue;
    return pre ? launch_two<T, true>(n, W, dinv, a, st) : launch_two<T, false>(n, W, dinv, a, st);
}

#define AGCA_INST(T)                                                                                       \
    template hipError_t launch_weights<T>(int, const double*, const uint16_t*, T*, float*, hipStream_t);    \
    template hipError_t launch_product7<T>(int, int, const T*, const T*, const T*, const T*, T*,           \
                                           const Sweep<T>&, hipStream_t);                                  \
    template hipError_t launch_two7<T>(bool, int, const T*, const T*, const Smooth2<T>&, hipStream_t);
AGCA_INST(double)
AGCA_INST(float)
#undef AGCA_INST

}  // namespace agca
