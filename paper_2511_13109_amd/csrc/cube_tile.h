// Device helpers shared by the element-loop kernels (k_apply.hip, k_smooth2.hip):
// neighbour exchange, coefficient loads and the workgroup -> tile mapping.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <utility>

#include "kuhn.h"

namespace agca {

// x neighbour exchange: DPP wave_shr:1, the value of the lane one to the left in the
// wavefront (0 for its first lane).  Tile rows are tw consecutive lanes and every
// wavefront starts a row, so the only lanes whose shifted-in value comes from another
// row are the rows' first lanes, the halo column, whose value is never used.
constexpr int kWaveShr1 = 0x138;
template <typename T>
__device__ __forceinline__ T shr1_row(T v) {
    constexpr int ctrl = kWaveShr1;
    if constexpr (sizeof(T) == 8) {
        const unsigned long long bits = __double_as_longlong(v);
        int lo = (int)(bits & 0xffffffffull);
        int hi = (int)(bits >> 32);
        lo = __builtin_amdgcn_update_dpp(0, lo, ctrl, 0xF, 0xF, true);
        hi = __builtin_amdgcn_update_dpp(0, hi, ctrl, 0xF, 0xF, true);
        return __longlong_as_double(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
    } else {
        int b = __float_as_int(v);
        b = __builtin_amdgcn_update_dpp(0, b, ctrl, 0xF, 0xF, true);
        return __int_as_float(b);
    }
}

// the value of the lane one to the right (0 for the last)
constexpr int kWaveShl1 = 0x130;
template <typename T>
__device__ __forceinline__ T shl1_row(T v) {
    if constexpr (sizeof(T) == 8) {
        const unsigned long long bits = __double_as_longlong(v);
        const int lo = __builtin_amdgcn_update_dpp(0, (int)(bits & 0xffffffffull), kWaveShl1, 0xF, 0xF, true);
        const int hi = __builtin_amdgcn_update_dpp(0, (int)(bits >> 32), kWaveShl1, 0xF, 0xF, true);
        return __longlong_as_double(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
    } else {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kWaveShl1, 0xF, 0xF, true));
    }
}

__device__ __forceinline__ float bf16_to_float(uint32_t bits16) { return __uint_as_float(bits16 << 16); }

// The six coefficients of a cell as loaded (in their storage type), decoded only when
// used: a select or conversion right after a load would make the wavefront wait for
// it at once.  AoS: three 16-byte (FP64), 8-byte (FP32) or 4-byte (BF16) loads.
template <typename NT>
struct RawNu;
template <>
struct RawNu<double> {
    double v[6];
    __device__ __forceinline__ void load(const double* __restrict__ p, int64_t stride) {
        if constexpr (AGCA_ELEM_SOA) {
#pragma unroll
            for (int s = 0; s < 6; ++s) v[s] = p[s * stride];
        } else {
            const double2* q = reinterpret_cast<const double2*>(p);
            const double2 a = q[0], b = q[1], c = q[2];
            v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y; v[4] = c.x; v[5] = c.y;
        }
    }
    template <typename T>
    __device__ __forceinline__ T get(int s) const { return T(v[s]); }
};
template <>
struct RawNu<float> {
    float v[6];
    __device__ __forceinline__ void load(const float* __restrict__ p, int64_t stride) {
        if constexpr (AGCA_ELEM_SOA) {
#pragma unroll
            for (int s = 0; s < 6; ++s) v[s] = p[s * stride];
        } else {
            const float2* q = reinterpret_cast<const float2*>(p);
            const float2 a = q[0], b = q[1], c = q[2];
            v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y; v[4] = c.x; v[5] = c.y;
        }
    }
    template <typename T>
    __device__ __forceinline__ T get(int s) const { return T(v[s]); }
};
template <>
struct RawNu<uint16_t> {
    uint32_t w[6];  // bf16 bits in the low half (SoA) or packed pairs in w[0..2] (AoS)
    __device__ __forceinline__ void load(const uint16_t* __restrict__ p, int64_t stride) {
        if constexpr (AGCA_ELEM_SOA) {
#pragma unroll
            for (int s = 0; s < 6; ++s) w[s] = p[s * stride];
        } else {
            const uint32_t* q = reinterpret_cast<const uint32_t*>(p);
            w[0] = q[0]; w[1] = q[1]; w[2] = q[2];
        }
    }
    template <typename T>
    __device__ __forceinline__ T get(int s) const {
        if constexpr (AGCA_ELEM_SOA) return T(bf16_to_float(w[s] & 0xffffu));
        const uint32_t x = w[s >> 1];
        return T(bf16_to_float((s & 1) ? (x >> 16) : (x & 0xffffu)));
    }
};

// Workgroup -> tile mapping.  Consecutive workgroups are dispatched round-robin
// to the 8 XCDs, each with its own L2; remapping the linear id so that every XCD
// receives one contiguous range of tiles (x fastest, then y, then z chunks)
// keeps the halo rows that neighbouring tiles share in the same L2.
// cols tile columns per z chunk, gz chunks (negative: no remapping)
__device__ __forceinline__ int tile_lin(int cols, int gz) {
    const int b = blockIdx.x;
    if (gz <= 0) return b;
    const int total = cols * gz;
    const int q = total >> 3, r = total & 7;
    const int xcd = b & 7, j = b >> 3;
    return xcd * q + min(xcd, r) + j;
}

// Global accesses of the z-marching kernels may go through buffer descriptors of one node or cell layer,
// formed per step by scalar instructions: a lane's address is one 32-bit offset, a load
// past the layer's end returns 0 and a store there is dropped.  Lanes outside the lattice
// or on its boundary therefore carry the offset kOut instead of selects and branches, and
// a layer outside the lattice has length 0.
constexpr uint32_t kOut = 0xf0000000u;
using Rsrc = __amdgpu_buffer_rsrc_t;
using u32x2 = uint32_t __attribute__((ext_vector_type(2)));
using u32x3 = uint32_t __attribute__((ext_vector_type(3)));
using u32x4 = uint32_t __attribute__((ext_vector_type(4)));
template <typename P>
__device__ __forceinline__ Rsrc layer_of(const P* p, bool inside, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<P*>(p), 0, inside ? (int)bytes : 0, 0x00027000);
}
template <typename T>
__device__ __forceinline__ T bload(Rsrc r, uint32_t off) {
    if constexpr (sizeof(T) == 8)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
    else
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
template <typename T>
__device__ __forceinline__ void bstore(Rsrc r, uint32_t off, T v) {
    if constexpr (sizeof(T) == 8)
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, off, 0, 0);
    else
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, off, 0, 0);
}
// The coarse correction, added to the iterate where a two-product pass stages it: fine node X
// takes half of e at the coarse nodes X/2 rounded down and up (k_vec.hip, Transfers).  Of the
// coarse level a tile of TX+1 x TY+1 fine nodes needs EX x EY nodes in each of two layers, which
// the workgroup keeps in LDS (layer m in buffer m & 1): fine layer f = 2m reads layer m, f = 2m+1
// layers m and m+1.  Layer m+1 is loaded in the step that stages f = 2m-1 and stored in the next one, a
// barrier after the last reads of layer m-1, whose buffer it takes.
template <int NC, typename T, int TX, int TY>
struct CoarseTile {
    static constexpr int EX = TX / 2 + 2, EY = TY / 2 + 2, EN = EX * EY;
    static_assert(EN <= 256 && EN <= TX * TY);
    using Tile = T[2][NC][EN];
    const T* e;
    int nc, x0, y0;
    // n: the fine level's; (X0, Y0): first fine node of the tile
    __device__ __forceinline__ void init(const T* e_, int n, int X0, int Y0) {
        e = e_;
        nc = n >> 1;
        x0 = X0 >> 1;
        y0 = Y0 >> 1;
    }
    // The next two are constants of a thread, for the caller to keep.
    // coarse nodes of the thread's fine nodes a and b: lower and upper one, 8 bits each
    __device__ __forceinline__ uint32_t slots(int xa, int ya, int xb, int yb) const {
        auto slot = [&](int X, int Y) { return (uint32_t)(((X >> 1) - x0) + EX * ((Y >> 1) - y0)); };
        return slot(xa, ya) | slot(xa + 1, ya + 1) << 8 | slot(xb, yb) << 16 | slot(xb + 1, yb + 1) << 24;
    }
    // offset in a coarse layer of the value that the thread loads (boundary values count 0)
    __device__ __forceinline__ uint32_t offset() const {
        const int r = threadIdx.x, x = x0 + r % EX, y = y0 + r / EX;
        return r < EN && x > 0 && x < nc && y > 0 && y < nc ? (uint32_t)(x + (nc + 1) * y) * (uint32_t)sizeof(T) : kOut;
    }
    // layer m's values of the thread (nothing is read unless `on`)
    __device__ __forceinline__ void load(int m, uint32_t at, bool on, T (&v)[NC]) const {
        // a coarse level (3 x 513^3 values at most) ends below 2^32 bytes
        const uint32_t n1 = (uint32_t)__builtin_amdgcn_readfirstlane(nc) + 1, layer = n1 * n1 * (uint32_t)sizeof(T);
#pragma unroll
        for (int c = 0; c < NC; ++c)
            v[c] = bload<T>(layer_of(reinterpret_cast<const char*>(e) + (c * n1 + (uint32_t)m) * layer, on && m > 0 && m < nc, layer), at);
    }
    __device__ __forceinline__ void store(Tile& es, int m, const T (&v)[NC]) const {
        if ((int)threadIdx.x < EN)
#pragma unroll
            for (int c = 0; c < NC; ++c) es[m & 1][c][threadIdx.x] = v[c];
    }
    // the correction at the thread's fine node k (0: a, 1: b) of layer f
    static __device__ __forceinline__ void value(const Tile& es, int f, int k, uint32_t slots, T (&out)[NC]) {
        const int lo = (slots >> (16 * k)) & 255, hi = (slots >> (16 * k + 8)) & 255;
#pragma unroll
        for (int c = 0; c < NC; ++c) out[c] = T(0.5) * (es[(f >> 1) & 1][c][lo] + es[((f + 1) >> 1) & 1][c][hi]);
    }
};

// Chunks of z layers: the count that minimises rounds x steps x time of a step.  A chunk of
// zc layers marches zc + 4 steps; a step with k workgroups on a compute unit takes about
// (3 + 4 k) / 7 of one with a single workgroup (129^3 FP32: 2.15 us for k = 1, 3.4 us for 2).
// Against sweeps of 1 to 43 chunks on the finest level (V-cycle, Chebyshev (2, 2)) the count
// is the best one at 65^3 and 129^3 in every form and precision (129^3 vector FP64 5 chunks 357 us, 4 / 10: 392 / 382;
// BF16/FP32 10 chunks 218, 9 / 5: 229 / 232; scalar FP64 10 chunks 118, 5: 120); at 257^3 7 chunks
// are best throughout (vector FP64 1856, chosen; BF16 983 against 1020 with the 8 chosen, FP32 1060 / 1090,
// scalar FP64 658 / 671 with 4, FP32 424 / 436 with 4).
inline int pick_chunks(int n, int64_t cols, int per_cu, int64_t cus) {
    int best = 1;
    double cost = -1.0;
    for (int gz = 1; gz <= n + 1; ++gz) {
        const int zc = (n + gz) / gz;
        if ((n + zc) / zc != gz) continue;  // the same chunk length with fewer chunks
        const int64_t wgs = cols * gz;
        const int64_t k = std::min<int64_t>(per_cu, (wgs + cus - 1) / cus);
        const int64_t rounds = (wgs + k * cus - 1) / (k * cus);
        const double c = (double)rounds * (zc + 4.5) * (3.0 + 4.0 * k);
        if (cost < 0.0 || c < cost) {
            cost = c;
            best = gz;
        }
    }
    return best;
}

// workgroups of a kernel that fit on a compute unit, and the compute units
template <typename K>
inline std::pair<int, int> workgroups_fit(K kernel, int threads) {
    int per_cu = 0, dev = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess ||
        hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || per_cu < 1 || cus < 1) {
        (void)hipGetLastError();
        return {1, 256};
    }
    return {per_cu, cus};
}

}  // namespace agca
