// mp_scan_index.hpp -- nearest-neighbour searches over a scan in walk order:
// its points, the boxes of every 64 of them, and the boxes of every 16 blocks.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mp_internal.hpp"
#include "mp_row.hpp"

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

// A box's order among the 16 of a row: its distance (rounded down by up to 15
// units in the last place, so that it bounds the points in it as before) and
// the lane; ~0 for none.
__device__ __forceinline__ uint32_t mp_box_key(bool in, const float4* b, const float3 p, int lane) {
    return in ? (__float_as_uint(mp_box_d2(b, p)) & ~15u) | (uint32_t)lane : ~0u;
}
