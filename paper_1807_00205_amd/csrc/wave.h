// Sorting by one wave in registers.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace sdf {

// The value of lane ^ j (j < 64, a power of two, known at compile time where
// the sort is unrolled): quad permutations (DPP) for 1 and 2, a swizzle
// within 32 lanes for 4 to 16, a permute for 32.
__device__ __forceinline__ uint32_t lane_xor(uint32_t v, uint32_t j) {
    switch (j) {
    case 1: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, false);  // [1,0,3,2]
    case 2: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, false);  // [2,3,0,1]
    case 4: return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, (4 << 10) | 0x1F);
    case 8: return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, (8 << 10) | 0x1F);
    case 16: return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, (16 << 10) | 0x1F);
    default: return (uint32_t)__shfl_xor((int)v, (int)j, 64);
    }
}

// Ascending bitonic sort of 64 E keys in registers, element e * 64 + lane.
template <class K, int E>
__device__ __forceinline__ void wave_sort_keys(K (&x)[E], uint32_t lane) {
#pragma unroll
    for (uint32_t k = 2; k <= 64u * E; k <<= 1) {
#pragma unroll
        for (uint32_t j = k >> 1; j > 0; j >>= 1) {
#pragma unroll
            for (int e = 0; e < E; e++) {
                if (j >= 64) {  // between registers: each pair once
                    const int f = e ^ (int)(j >> 6);
                    if (f < e) continue;
                    const bool up = ((uint32_t)(e * 64) & k) == 0;
                    const K lo = x[e] < x[f] ? x[e] : x[f], hi = x[e] < x[f] ? x[f] : x[e];
                    x[e] = up ? lo : hi;
                    x[f] = up ? hi : lo;
                } else {
                    K y;
                    if constexpr (sizeof(K) == 8)
                        y = ((K)lane_xor((uint32_t)(x[e] >> 32), j) << 32) | lane_xor((uint32_t)x[e], j);
                    else
                        y = lane_xor(x[e], j);
                    const bool up = (((uint32_t)(e * 64) | (lane & 63)) & k) == 0;
                    const bool lower = (lane & j) == 0;
                    const K lo = x[e] < y ? x[e] : y, hi = x[e] < y ? y : x[e];
                    x[e] = lower == up ? lo : hi;
                }
            }
        }
    }
}

}  // namespace sdf
