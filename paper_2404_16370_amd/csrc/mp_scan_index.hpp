// mp_scan_index.hpp -- nearest-neighbour searches over a scan in walk order:
// its points, the boxes of every 64 of them, and the boxes of every 16 blocks.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mp_internal.hpp"

// FP32 squared distance of the searches (the residual gate's fma order)
__device__ __forceinline__ float mp_point_d2(const float4 c, const float3 p) {
    const float dx = c.x - p.x, dy = c.y - p.y, dz = c.z - p.z;
    return __builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, dz * dz));
}

// Lower bound of mp_point_d2 over the points of a box (lower corner, upper
// corner).  Rounding is monotone, so the bound computed with the same
// operations from the nearest face never exceeds the computed distance of a
// point inside: a box above a search's bound holds nothing that the search
// would take, not even an equal distance.
__device__ __forceinline__ float mp_box_d2(const float4* __restrict__ b, const float3 p) {
    const float4 lo = b[0], hi = b[1];
    const float dx = fmaxf(fmaxf(lo.x - p.x, p.x - hi.x), 0.0f);
    const float dy = fmaxf(fmaxf(lo.y - p.y, p.y - hi.y), 0.0f);
    const float dz = fmaxf(fmaxf(lo.z - p.z, p.z - hi.z), 0.0f);
    return __builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, dz * dz));
}

// value of the lane `rot` places on in this lane's row of 16
template <int ROT>
__device__ __forceinline__ uint32_t mp_row_ror(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x120 + ROT, 0xF, 0xF, true);
}

// maximum over the row of 16 lanes (every lane of the wave active)
__device__ __forceinline__ float mp_row_max(float v) {
    v = fmaxf(v, __uint_as_float(mp_row_ror<8>(__float_as_uint(v))));
    v = fmaxf(v, __uint_as_float(mp_row_ror<4>(__float_as_uint(v))));
    v = fmaxf(v, __uint_as_float(mp_row_ror<2>(__float_as_uint(v))));
    return fmaxf(v, __uint_as_float(mp_row_ror<1>(__float_as_uint(v))));
}

// the votes of this lane's row of 16 (every lane of the wave active)
__device__ __forceinline__ uint32_t mp_row_ballot(bool p) {
    return (uint32_t)(__ballot(p) >> (threadIdx.x & 48)) & 0xFFFFu;
}
