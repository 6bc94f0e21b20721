// Device helpers shared by the element-loop kernels (k_apply.hip, k_smooth2.hip):
// neighbour exchange, coefficient loads and the workgroup -> tile mapping.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

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

}  // namespace agca
