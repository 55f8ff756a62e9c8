// mp_place.hpp -- where a kernel of a filter may write (host code only).
#pragma once
#include <hip/hip_runtime_api.h>

// A kernel stores straight into memory of its filter's own device, or into
// managed memory.  Memory of another device (which it could only reach with
// peer access) and host memory are written by copies.
inline bool mp_in_place(const hipPointerAttribute_t& a, int device) {
    return a.type == hipMemoryTypeManaged || (a.type == hipMemoryTypeDevice && a.device == device);
}
