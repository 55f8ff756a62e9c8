// mp_row.hpp -- exchanges within a row of 16 lanes (every lane of the wave active).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

// value of the lane `rot` places on in this lane's row of 16
template <int ROT>
__device__ __forceinline__ uint32_t mp_row_ror(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x120 + ROT, 0xF, 0xF, true);
}

// maximum over the row of 16 lanes
__device__ __forceinline__ float mp_row_max(float v) {
    v = fmaxf(v, __uint_as_float(mp_row_ror<8>(__float_as_uint(v))));
    v = fmaxf(v, __uint_as_float(mp_row_ror<4>(__float_as_uint(v))));
    v = fmaxf(v, __uint_as_float(mp_row_ror<2>(__float_as_uint(v))));
    return fmaxf(v, __uint_as_float(mp_row_ror<1>(__float_as_uint(v))));
}

// minimum over the row
__device__ __forceinline__ float mp_row_min(float v) {
    v = fminf(v, __uint_as_float(mp_row_ror<8>(__float_as_uint(v))));
    v = fminf(v, __uint_as_float(mp_row_ror<4>(__float_as_uint(v))));
    v = fminf(v, __uint_as_float(mp_row_ror<2>(__float_as_uint(v))));
    return fminf(v, __uint_as_float(mp_row_ror<1>(__float_as_uint(v))));
}

// the votes of this lane's row of 16
__device__ __forceinline__ uint32_t mp_row_ballot(bool p) {
    return (uint32_t)(__ballot(p) >> (threadIdx.x & 48)) & 0xFFFFu;
}

__device__ __forceinline__ uint32_t mp_row_min_u32(uint32_t v) {
    v = min(v, mp_row_ror<8>(v));
    v = min(v, mp_row_ror<4>(v));
    v = min(v, mp_row_ror<2>(v));
    return min(v, mp_row_ror<1>(v));
}

template <int ROT>
__device__ __forceinline__ uint64_t mp_row_min_step(uint64_t v) {
    const uint64_t o = ((uint64_t)mp_row_ror<ROT>((uint32_t)(v >> 32)) << 32) | mp_row_ror<ROT>((uint32_t)v);
    return o < v ? o : v;
}

// minimum over the row
__device__ __forceinline__ uint64_t mp_row_min_u64(uint64_t v) {
    return mp_row_min_step<1>(mp_row_min_step<2>(mp_row_min_step<4>(mp_row_min_step<8>(v))));
}

// value of the lane before this one in the row; `first` for the row's lane 0
__device__ __forceinline__ uint64_t mp_row_shr(uint64_t v, uint64_t first) {
    const int lo = __builtin_amdgcn_update_dpp((int)(uint32_t)first, (int)(uint32_t)v, 0x111, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(uint32_t)(first >> 32), (int)(uint32_t)(v >> 32), 0x111, 0xF, 0xF, false);
    return ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo;
}
