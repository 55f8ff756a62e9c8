// mp_lsh.hpp -- the bucket code of a particle (Eq. 9), for the kernels that
// leave it: k_lsh, and k_svgd for the iteration that follows.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mp_det.hpp"
#include "mp_internal.hpp"

struct LshArgs {
    const float4* __restrict__ poses;
    uint32_t* __restrict__ codes;     // particle order
    uint32_t* __restrict__ keys;      // the bucket sort's input keys (a copy of codes)
    int32_t* __restrict__ idx;        // the bucket sort's input values (0..n-1)
    float* __restrict__ tlsh;
    int32_t n;
    uint32_t mask, frame, it;
    float ar, at, sl;
    int32_t coupled;                  // tangent: 0 decoupled, 1 coupled SE(3) log
    float lo[3], hi[3];
    uint64_t seed;
    const StepDyn* __restrict__ dyn;   // captured step: frame from here
    int32_t* flags;                    // the step's counters to clear, or null
    uint64_t* stamp;                   // stage clock, or null
};
LshArgs mp_lsh_args(mp_filter f, uint32_t frame, uint32_t it);

// T^LSH is the same for every particle: one lane of a workgroup draws it (and one records it)
__device__ __forceinline__ void lsh_draw(const LshArgs& A, float* sL, bool record) {
    mpdet::quat q0;
    float3 t0;
    mpdet::random_pose(A.seed, 0u, A.frame, A.it, mpdet::PURPOSE_TLSH, A.lo, A.hi, q0, t0);
    sL[0] = q0.w; sL[1] = q0.x; sL[2] = q0.y; sL[3] = q0.z;
    sL[4] = t0.x; sL[5] = t0.y; sL[6] = t0.z; sL[7] = 0.0f;
    if (record)
        for (int k = 0; k < 8; ++k) A.tlsh[k] = sL[k];
}

// the code of particle i at pose (q4, t4)
__device__ __forceinline__ void lsh_code(const LshArgs& A, const float* sL, int i, const float4 q4, const float4 t4) {
    const mpdet::quat qL{sL[0], sL[1], sL[2], sL[3]};
    const float3 tL = make_float3(sL[4], sL[5], sL[6]);
    const mpdet::quat qi{q4.x, q4.y, q4.z, q4.w};
    float3 om, u;
    if (A.coupled) {
        mpdet::se3_between(qL, tL, qi, make_float3(t4.x, t4.y, t4.z), om, u);
    } else {
        const mpdet::quat qr = mpdet::qmul(mpdet::qconj(qL), qi);
        float w, sc;
        om = mpdet::qlog(qr, w, sc);
        const mpdet::mat3 RL = mpdet::qmat(qL);
        u = mpdet::rot_t(RL, make_float3(t4.x - tL.x, t4.y - tL.y, t4.z - tL.z));
    }
    float z[6];
    mpdet::gauss6(A.seed, (uint32_t)i, A.frame, A.it, mpdet::PURPOSE_LSH, z);
    int32_t c[6];
    c[0] = mpdet::floor_i32(A.ar * om.x + A.sl * z[0]);
    c[1] = mpdet::floor_i32(A.ar * om.y + A.sl * z[1]);
    c[2] = mpdet::floor_i32(A.ar * om.z + A.sl * z[2]);
    c[3] = mpdet::floor_i32(A.at * u.x + A.sl * z[3]);
    c[4] = mpdet::floor_i32(A.at * u.y + A.sl * z[4]);
    c[5] = mpdet::floor_i32(A.at * u.z + A.sl * z[5]);
    const uint32_t code = mpdet::hash6(c) & A.mask;
    A.codes[i] = code;
    A.keys[i] = code;
    A.idx[i] = i;
}
