// Wave64 / workgroup prefix sums used by the sort and emission kernels.
#pragma once
#include <hip/hip_runtime.h>

namespace gft {

__device__ __forceinline__ int lane_id() { return __lane_id(); }

template <typename T>
__device__ __forceinline__ T wave_inclusive_scan(T x) {
    const int lane = lane_id();
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        T y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    return x;
}

// 32-bit integers: row shifts and row broadcasts of the lanes (DPP) in place
// of six trips through LDS.
template <>
__device__ __forceinline__ uint32_t wave_inclusive_scan<uint32_t>(uint32_t x) {
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);   // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);   // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);   // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);   // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);   // row_bcast:15, rows 1 and 3
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);   // row_bcast:31, rows 2 and 3
    return x;
}

template <typename T>
__device__ __forceinline__ T wave_reduce_sum(T x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}

// Exclusive scan over a workgroup of NT threads (NT multiple of 64, <= 1024).
// `scratch` must hold NT/64 elements of T.  Returns the exclusive prefix
// of the calling thread; *total receives the workgroup sum.  Contains
// barriers: every thread of the workgroup must call it.
template <typename T, int NT>
__device__ __forceinline__ T block_exclusive_scan(T x, T* scratch, T* total) {
    constexpr int NW = NT / 64;
    const int lane = lane_id();
    const int wave = threadIdx.x / 64;
    T inc = wave_inclusive_scan(x);
    if (lane == 63) scratch[wave] = inc;
    __syncthreads();
    T before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const T v = scratch[w];
        before += w < wave ? v : T(0);
        all += v;
    }
    *total = all;
    __syncthreads();
    return before + inc - x;
}

}  // namespace gft
