// odometry.hip -- GICP scan-to-scan odometry (Sec. III-B): the sensor motion
// dT between the previous and the current scan, and its covariance from the
// Hessian of the match, the inputs of the prediction step (Eq. 1); GICP after
// Segal et al. (2009).
//
// Source = the current scan (points mu_k, covariances S_k), target = the
// previous scan (points q_j, covariances T_j); dT maps current-frame points
// into the previous frame (T_t = T_{t-1} dT).  At pose (R, t):
//   p_k = R mu_k + t (FP32, the filter's transform program),
//   j(k) = argmin_j |q_j - p_k|^2 (FP32, the residual gate's fma order,
//          ties to the lower index), an inlier iff that is <= d_max^2;
//   e = q_j - p_k; in the body frame e_b = R^T e,
//   C_b = R^T T_j R + S_k, Omega_b = C_b^-1, J_b = [[mu]x, -I]:
//   H += J_b^T Omega_b J_b, b += J_b^T Omega_b e_b, cost += e_b^T Omega_b e_b
//   (FP32 per point, FP64 sums in a fixed order).
// Each iteration: psi = -(H + diag(lam_rel H_ii + lam_abs))^-1 b (FP64),
// dT <- dT exp(psi) (FP64 pose, FP32 copy for the next evaluation).  After
// the last update the terms are evaluated once more: Sigma^dT = scale H^-1.
//
// One launch per iteration.  Every workgroup adds the sums that the
// workgroups of the launch before left and takes the step itself (the same
// operations in the same order, so all hold the same pose); then it matches
// its source points, 16 lanes a point, through the spatial index of the
// previous scan (boxes of 64 and of 1024 of its points), starting from the
// point's match of the iteration before: a box farther away than the best
// distance so far, or than d_max, holds no better match.  Then one lane per
// source point forms its terms, and the workgroup leaves their FP64 sums,
// added in a fixed order.
//
// What bounds it: latency (the sums and the step's FP64 chain, about 3 us,
// then the dependent loads of the search).  An iteration takes 16 us on
// 8192-point scans and 51 us on 65,536-point ones; searching all targets for
// every point, with the step and the terms in launches of their own, took 36
// and 820 us.  The first two iterations, whose matches of the iteration before
// are missing or far off, take the boxes nearest first (65,536 points: 131 and
// 81 -> 59 and 60 us); for the later ones finding the nearest box costs more
// than the few others that are still below the bound (51 -> 57 us).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>

#include "megapf.h"
#include "mp_det.hpp"
#include "mp_internal.hpp"
#include "mp_scan_index.hpp"

namespace {

constexpr int kOThreads = 512;
constexpr int kOLanes = 16;                        // lanes per source point in the search
constexpr int kOSlots = kOThreads / kOLanes;       // source points matched at a time
constexpr int kOParts = 512;                       // most workgroups of a launch
constexpr int kORounds = 4;                        // most rounds of a workgroup
constexpr int kOTerms = 29;                        // H (21), b (6), cost, inlier count per source point
constexpr int kOBlocks = 65536 / kScanBlock;       // boxes of the largest scan
constexpr int kOSum = 16;                          // every sum is taken in this many parts, then over them
static_assert(kOParts * kORounds * kOSlots >= 65536, "the largest scan");
static_assert(kOTerms * kOSum <= kOThreads, "one thread per part of a sum");

__device__ __forceinline__ float3 odo_point(const float* pose, const mpdet::mat3& Rm, const float4 r) {
    return mpdet::xform(Rm.m, make_float3(pose[4], pose[5], pose[6]), make_float3(r.x, r.y, r.z));
}

struct OdoArgs {
    ScanIndex T;                       // the previous scan's index
    const float4* __restrict__ trec;   // its records, caller order (3 float4 per point)
    const float4* __restrict__ swalk;  // the current scan's records in its index's order
    const float4* __restrict__ spts;   // and its points with their caller index
    int32_t* nn;                       // ns, caller order: target index or -1 (read and rewritten by each iteration)
    const double* __restrict__ part_in;   // the iteration before: [kOTerms][kOParts] workgroup sums
    double* __restrict__ part_out;
    const double* __restrict__ pose_in;   // and its pose (7)
    double* __restrict__ pose_out;
    double init[7];                    // first iteration: the starting pose
    double lam_rel, lam_abs;
    int32_t ns, nparts, rounds, first;
    float dmax2;
};

// The GICP terms of one source point given its nearest target (zero for an
// outlier); t[28] is the inlier count.
__device__ __forceinline__ void odo_point_terms(const OdoArgs& A, const float* pose, const mpdet::mat3& Rm,
                                                const int ws, const int bj, float t[kOTerms]) {
    const float4 s0 = A.swalk[3 * ws];
    const float3 mu = make_float3(s0.x, s0.y, s0.z);
    const float3 p = odo_point(pose, Rm, s0);
    const float4 t0 = A.trec[3 * bj], t1 = A.trec[3 * bj + 1], t2 = A.trec[3 * bj + 2];
    const float4 s1 = A.swalk[3 * ws + 1], s2 = A.swalk[3 * ws + 2];
    const float3 eb = mpdet::rot_t(Rm, make_float3(t0.x - p.x, t0.y - p.y, t0.z - p.z));
    // R^T T R: columns of T R, then R^T times them
    const float T[3][3] = {{t0.w, t1.x, t1.y}, {t1.x, t1.z, t1.w}, {t1.y, t1.w, t2.x}};
    float TR[3][3], C[3][3];
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c)
            TR[r][c] = T[r][0] * Rm.m[c] + T[r][1] * Rm.m[3 + c] + T[r][2] * Rm.m[6 + c];
    const float S[3][3] = {{s0.w, s1.x, s1.y}, {s1.x, s1.z, s1.w}, {s1.y, s1.w, s2.x}};
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c)
            C[r][c] = Rm.m[r] * TR[0][c] + Rm.m[3 + r] * TR[1][c] + Rm.m[6 + r] * TR[2][c] + S[r][c];
    // Omega_b = C_b^-1 (adjugate of the symmetrised matrix)
    const float c00 = C[0][0], c01 = 0.5f * (C[0][1] + C[1][0]), c02 = 0.5f * (C[0][2] + C[2][0]);
    const float c11 = C[1][1], c12 = 0.5f * (C[1][2] + C[2][1]), c22 = C[2][2];
    const float i00 = c11 * c22 - c12 * c12, i01 = c02 * c12 - c01 * c22, i02 = c01 * c12 - c02 * c11;
    const float i11 = c00 * c22 - c02 * c02, i12 = c01 * c02 - c00 * c12, i22 = c00 * c11 - c01 * c01;
    const float rd = 1.0f / (c00 * i00 + c01 * i01 + c02 * i02);
    const float O[3][3] = {{i00 * rd, i01 * rd, i02 * rd}, {i01 * rd, i11 * rd, i12 * rd}, {i02 * rd, i12 * rd, i22 * rd}};
    const float e[3] = {eb.x, eb.y, eb.z};
    float w[3];
    for (int r = 0; r < 3; ++r) w[r] = O[r][0] * e[0] + O[r][1] * e[1] + O[r][2] * e[2];
    // J_b = [[mu]x, -I]
    const float J[3][6] = {{0.0f, -mu.z, mu.y, -1.0f, 0.0f, 0.0f},
                           {mu.z, 0.0f, -mu.x, 0.0f, -1.0f, 0.0f},
                           {-mu.y, mu.x, 0.0f, 0.0f, 0.0f, -1.0f}};
    float OJ[3][6];
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 6; ++c) OJ[r][c] = O[r][0] * J[0][c] + O[r][1] * J[1][c] + O[r][2] * J[2][c];
    int q = 0;
    for (int r = 0; r < 6; ++r)
        for (int c = r; c < 6; ++c) t[q++] = J[0][r] * OJ[0][c] + J[1][r] * OJ[1][c] + J[2][r] * OJ[2][c];
    for (int r = 0; r < 6; ++r) t[21 + r] = J[0][r] * w[0] + J[1][r] * w[1] + J[2][r] * w[2];
    t[27] = e[0] * w[0] + e[1] * w[1] + e[2] * w[2];
    t[28] = 1.0f;
}

// The sums of the workgroups of one launch: every term in kOSum parts, then
// over the parts (a fixed order, the same in every workgroup).
__device__ __forceinline__ void odo_total(const double* __restrict__ part, int nparts, double (*run)[kOSum],
                                          double* tot) {
    if (threadIdx.x < kOTerms * kOSum) {
        const int m = threadIdx.x / kOSum, c = threadIdx.x % kOSum;
        double acc = 0.0;
        constexpr int kFly = 16;   // loads in flight together
        for (int g0 = c; g0 < nparts; g0 += kFly * kOSum) {
            double v[kFly];
#pragma unroll
            for (int u = 0; u < kFly; ++u) {
                const int g = g0 + u * kOSum;
                v[u] = part[m * kOParts + min(g, nparts - 1)];
            }
#pragma unroll
            for (int u = 0; u < kFly; ++u) acc += g0 + u * kOSum < nparts ? v[u] : 0.0;
        }
        run[m][c] = acc;
    }
    __syncthreads();
    if (threadIdx.x < kOTerms) {
        double acc = 0.0;
        for (int c = 0; c < kOSum; ++c) acc += run[threadIdx.x][c];
        tot[threadIdx.x] = acc;
    }
    __syncthreads();
}

// x = -(H + diag(lam_rel H_ii + lam_abs))^-1 b by an L D L^T factorisation;
// false if a pivot is not positive
__device__ __forceinline__ bool odo_solve(const double* H, const double* b, double lam_rel, double lam_abs,
                                          double x[6]) {
    double L[6][6], D[6], inv[6];
    bool ok = true;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        const double h = H[j * 6 - j * (j - 1) / 2];   // H_jj of the packed upper triangle
        double d = h + (lam_rel * h + lam_abs);
#pragma unroll
        for (int k = 0; k < j; ++k) d -= L[j][k] * L[j][k] * D[k];
        ok = ok && d > 0.0;
        D[j] = d;
        inv[j] = 1.0 / d;
#pragma unroll
        for (int i = j + 1; i < 6; ++i) {
            double t = H[j * 6 - j * (j - 1) / 2 + (i - j)];
#pragma unroll
            for (int k = 0; k < j; ++k) t -= L[i][k] * L[j][k] * D[k];
            L[i][j] = t * inv[j];
        }
    }
    double y[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        double t = -b[i];
#pragma unroll
        for (int k = 0; k < i; ++k) t -= L[i][k] * y[k];
        y[i] = t;
    }
#pragma unroll
    for (int i = 5; i >= 0; --i) {
        double t = y[i] * inv[i];
#pragma unroll
        for (int k = i + 1; k < 6; ++k) t -= L[k][i] * x[k];
        x[i] = t;
    }
    return ok;
}

// SE(3) exponential of [omega; v] (FP64): unit quaternion + translation V v,
// V = I + A w^ + B w^2
__device__ void se3_exp_d(const double xi[6], double T[7]) {
    const double* w = xi;
    const double* v = xi + 3;
    const double th2 = w[0] * w[0] + w[1] * w[1] + w[2] * w[2];
    double A, B, hs, hc;   // (1 - cos)/th^2, (th - sin)/th^3, sin(th/2)/th, cos(th/2)
    if (th2 < 0.25) {      // Taylor series: the first term left out is below 1e-17 of the sum
        const double h2 = 0.25 * th2;   // (th/2)^2
        double s = 1.0, c = 1.0, b = 1.0;
#pragma unroll
        for (int n = 8; n >= 1; --n) {
            const double e = 2.0 * n;
            s = 1.0 - (s * h2) * (1.0 / (e * (e + 1.0)));
            c = 1.0 - (c * h2) * (1.0 / (e * (e - 1.0)));
            b = 1.0 - (b * th2) * (1.0 / ((e + 2.0) * (e + 3.0)));
        }
        hs = 0.5 * s;
        hc = c;
        A = 0.5 * s * s;
        B = b * (1.0 / 6.0);
    } else {
        const double th = sqrt(th2);
        A = (1.0 - cos(th)) / th2;
        B = (th - sin(th)) / (th2 * th);
        hs = sin(0.5 * th) / th;
        hc = cos(0.5 * th);
    }
    T[0] = hc;
    T[1] = hs * w[0];
    T[2] = hs * w[1];
    T[3] = hs * w[2];
    const double c1[3] = {w[1] * v[2] - w[2] * v[1], w[2] * v[0] - w[0] * v[2], w[0] * v[1] - w[1] * v[0]};
    const double c2[3] = {w[1] * c1[2] - w[2] * c1[1], w[2] * c1[0] - w[0] * c1[2], w[0] * c1[1] - w[1] * c1[0]};
    for (int k = 0; k < 3; ++k) T[4 + k] = v[k] + A * c1[k] + B * c2[k];
}

// P <- P exp(psi) with the damped step of the sums `tot`
__device__ void odo_step(const double* tot, double lam_rel, double lam_abs, const double* P, double out[7]) {
    double psi[6];
    if (!odo_solve(tot, tot + 21, lam_rel, lam_abs, psi))
        for (int m = 0; m < 6; ++m) psi[m] = 0.0;
    double D[7];
    se3_exp_d(psi, D);
    // Hamilton product and P's rotation applied to D's translation
    const double q[4] = {P[0] * D[0] - P[1] * D[1] - P[2] * D[2] - P[3] * D[3],
                         P[0] * D[1] + P[1] * D[0] + P[2] * D[3] - P[3] * D[2],
                         P[0] * D[2] - P[1] * D[3] + P[2] * D[0] + P[3] * D[1],
                         P[0] * D[3] + P[1] * D[2] - P[2] * D[1] + P[3] * D[0]};
    const double w = P[0], x = P[1], y = P[2], z = P[3];
    const double R[9] = {1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                         2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                         2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)};
    const double nq = sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
    for (int a = 0; a < 4; ++a) out[a] = q[a] / nq;
    for (int a = 0; a < 3; ++a) out[4 + a] = P[4 + a] + R[3 * a] * D[4] + R[3 * a + 1] * D[5] + R[3 * a + 2] * D[6];
}

__device__ __forceinline__ uint64_t odo_key(float d2, int32_t j) {   // d2 >= +0: its bits order as the values do
    return ((uint64_t)__float_as_uint(d2) << 32) | (uint32_t)j;
}

template <bool NEAREST>   // boxes nearest first, or in index order
__global__ __launch_bounds__(kOThreads) void k_odo_iter(OdoArgs A) {
    __shared__ double run[kOTerms][kOSum];
    __shared__ double tot[kOTerms];
    __shared__ float pose[8];
    __shared__ int32_t match[kOSlots * kORounds];
    __shared__ float tt[kOTerms][kOSlots * kORounds];
    __shared__ float4 box[2 * kOBlocks];                 // the boxes of the previous scan's index
    __shared__ float4 super[2 * (kOBlocks / kScanFan)];
    const int grp = threadIdx.x / kOLanes, gl = threadIdx.x % kOLanes;
    const int w0 = blockIdx.x * A.rounds * kOSlots;
    // the boxes are requested with the sums of the launch before and kept
    // after those have arrived
    constexpr int kPre = 2 * kOBlocks / kOThreads;
    float4 pre[kPre], pre_s;
#pragma unroll
    for (int u = 0; u < kPre; ++u) pre[u] = A.T.box[min((int)threadIdx.x + u * kOThreads, 2 * A.T.blocks - 1)];
    pre_s = A.T.super[min((int)threadIdx.x, 2 * A.T.supers - 1)];
    // the pose of this iteration
    if (!A.first) odo_total(A.part_in, A.nparts, run, tot);
#pragma unroll
    for (int u = 0; u < kPre; ++u)
        if ((int)threadIdx.x + u * kOThreads < 2 * A.T.blocks) box[threadIdx.x + u * kOThreads] = pre[u];
    if ((int)threadIdx.x < 2 * A.T.supers) super[threadIdx.x] = pre_s;
    if (threadIdx.x == 0) {
        double P[7];
        if (A.first) {
            for (int a = 0; a < 7; ++a) P[a] = A.init[a];
        } else {
            double in[7];
            for (int a = 0; a < 7; ++a) in[a] = A.pose_in[a];
            odo_step(tot, A.lam_rel, A.lam_abs, in, P);
        }
        for (int a = 0; a < 7; ++a) pose[a] = (float)P[a];
        pose[7] = 0.0f;
        if (blockIdx.x == 0)
            for (int a = 0; a < 7; ++a) A.pose_out[a] = P[a];
    }
    __syncthreads();
    const mpdet::mat3 Rm = mpdet::qmat(mpdet::quat{pose[0], pose[1], pose[2], pose[3]});
    // matches
#pragma unroll 1
    for (int r = 0; r < A.rounds; ++r) {
        const int w = w0 + r * kOSlots + grp;
        const bool active = w < A.ns;   // uniform over the point's lanes
        const float4 sp = A.spts[active ? w : 0];
        const int k = __float_as_int(sp.w);
        const float3 p = odo_point(pose, Rm, sp);
        // below this key a candidate is taken: within d_max, then better than the best so far
        uint64_t best = odo_key(A.dmax2, 0x7FFFFFFF);
        const uint64_t none = best;
        if (!A.first && active) {
            const int j = A.nn[k];
            if (j >= 0) {
                const uint64_t key = odo_key(mp_point_d2(A.trec[3 * j], p), j);
                best = key < best ? key : best;
            }
        }
        float bound = __uint_as_float((uint32_t)(best >> 32));
        // a block of a row's choice (if any) against its point
        const auto visit = [&](bool go, int blk) {
            const int q0 = go ? blk * kScanBlock + gl : A.T.n;
            float4 c[kScanBlock / kOLanes];
#pragma unroll
            for (int u = 0; u < kScanBlock / kOLanes; ++u) c[u] = A.T.pts[min(q0 + kOLanes * u, A.T.n - 1)];
#pragma unroll
            for (int u = 0; u < kScanBlock / kOLanes; ++u) {
                const uint64_t key = odo_key(mp_point_d2(c[u], p), __float_as_int(c[u].w));
                if (q0 + kOLanes * u < A.T.n && key < best) best = key;
            }
            best = mp_row_min_u64(best);
            bound = __uint_as_float((uint32_t)(best >> 32));
        };
        const int batches = (A.T.supers + kOLanes - 1) / kOLanes;
        if (NEAREST) {
            int batch = min(w / (kScanBlock * kScanFan * kOLanes), batches - 1);   // where its match likely is
            for (int b = 0; b < batches; ++b, batch = batch + 1 < batches ? batch + 1 : 0) {
                const int sup = batch * kOLanes + gl;
                uint32_t sk = mp_box_key(active && sup < A.T.supers, super + 2 * min(sup, A.T.supers - 1), p, gl);
                for (;;) {
                    const uint32_t su = mp_row_min_u32(sk);
                    const bool go = su != ~0u && __uint_as_float(su & ~15u) <= bound;
                    if (!__any(go)) break;
                    if ((su & 15u) == (uint32_t)gl) sk = ~0u;
                    const int blk0 = (batch * kOLanes + (int)(su & 15u)) * kScanFan;
                    const int blk = blk0 + gl;
                    uint32_t bk = mp_box_key(go && blk < A.T.blocks, box + 2 * min(blk, A.T.blocks - 1), p, gl);
                    for (;;) {
                        const uint32_t bl = mp_row_min_u32(bk);
                        const bool gob = bl != ~0u && __uint_as_float(bl & ~15u) <= bound;
                        if (!__any(gob)) break;
                        if ((bl & 15u) == (uint32_t)gl) bk = ~0u;
                        visit(gob, blk0 + (int)(bl & 15u));
                    }
                }
            }
        } else {
            for (int s0 = 0; s0 < A.T.supers; s0 += kOLanes) {
                const int sup = s0 + gl;
                uint32_t sm = mp_row_ballot(active && sup < A.T.supers &&
                                            mp_box_d2(super + 2 * min(sup, A.T.supers - 1), p) <= bound);
                while (__any(sm != 0)) {
                    const int su = s0 + (sm ? __builtin_ctz(sm) : 0);
                    const int blk = su * kScanFan + gl;
                    uint32_t bm = mp_row_ballot(sm != 0 && blk < A.T.blocks &&
                                                mp_box_d2(box + 2 * min(blk, A.T.blocks - 1), p) <= bound);
                    sm &= sm - 1;
                    while (__any(bm != 0)) {
                        visit(bm != 0, su * kScanFan + (bm ? __builtin_ctz(bm) : 0));
                        bm &= bm - 1;
                    }
                }
            }
        }
        if (gl == 0) {
            const int j = best == none ? -1 : (int)(uint32_t)best;
            match[r * kOSlots + grp] = active ? j : -1;
            if (active) A.nn[k] = j;
        }
    }
    __syncthreads();
    // terms, one lane per point
    const int np = A.rounds * kOSlots;
    if ((int)threadIdx.x < np) {
        float t[kOTerms];
        for (int m = 0; m < kOTerms; ++m) t[m] = 0.0f;
        const int j = match[threadIdx.x];
        if (j >= 0) odo_point_terms(A, pose, Rm, w0 + threadIdx.x, j, t);
        for (int m = 0; m < kOTerms; ++m) tt[m][threadIdx.x] = t[m];
    }
    __syncthreads();
    if (threadIdx.x < kOTerms * kOSum) {
        const int m = threadIdx.x / kOSum, c = threadIdx.x % kOSum;
        double acc = 0.0;
        for (int i = c; i < np; i += kOSum) acc += (double)tt[m][i];
        run[m][c] = acc;
    }
    __syncthreads();
    if (threadIdx.x < kOTerms) {
        double acc = 0.0;
        for (int c = 0; c < kOSum; ++c) acc += run[threadIdx.x][c];
        A.part_out[threadIdx.x * kOParts + blockIdx.x] = acc;
    }
}

// The final sums and the covariance: out = pose (7, then 0), H 21, b 6, cost,
// inliers, covariance 36, ok.
__global__ __launch_bounds__(kOThreads) void k_odo_final(const double* __restrict__ part, int nparts,
                                                         const double* __restrict__ pose, double cov_scale,
                                                         double* __restrict__ out) {
    __shared__ double run[kOTerms][kOSum];
    __shared__ double tot[kOTerms];
    odo_total(part, nparts, run, tot);
    if (threadIdx.x < 8) out[threadIdx.x] = threadIdx.x < 7 ? pose[threadIdx.x] : 0.0;
    if (threadIdx.x < kOTerms) out[8 + threadIdx.x] = tot[threadIdx.x];
    // Sigma = scale H^-1: column j solves H x = e_j (the undamped solve with b = -e_j)
    if (threadIdx.x < 6) {
        double e[6], x[6];
        for (int m = 0; m < 6; ++m) e[m] = m == (int)threadIdx.x ? -1.0 : 0.0;
        const bool ok = odo_solve(tot, e, 0.0, 0.0, x);
        for (int m = 0; m < 6; ++m) out[8 + 29 + 6 * m + threadIdx.x] = ok ? cov_scale * x[m] : 0.0;
        if (threadIdx.x == 0) out[8 + 65] = ok ? 1.0 : 0.0;
    }
}

}  // namespace

extern "C" void mp_odometry_default_params(mp_odometry_params* p) {
    if (!p) return;
    p->iterations = 20;
    p->d_max = 1.0f;
    p->lambda_rel = 1e-3f;
    p->lambda_abs = 1e-6f;
    p->cov_scale = 1.0f;
}

mp_status mp_guarded_call(const char* where, void (*fn)(void*), void* ctx);

namespace {
struct OdoCall {
    mp_filter f;
    const mp_odometry_params* p;
    const float* init;
    float* dT_out;
    float* cov_out;
    mp_odometry_result* res;
    hipStream_t s;
    char* scratch;   // device address of the fixed work area, or null: the filter's buffers
};

// Layout of the work area: matches, workgroup sums of two iterations, the
// poses of two iterations, the results.
constexpr size_t kNoAllocScan = 16384;   // largest current scan of mp_odometry_noalloc
constexpr size_t kPartBytes = sizeof(double) * kOTerms * kOParts;
constexpr size_t kOutDoubles = 8 + 66;
constexpr size_t kWorkBytes = 2 * kPartBytes + sizeof(double) * (16 + kOutDoubles);   // all but the matches
constexpr size_t kScrWork = sizeof(int32_t) * kNoAllocScan;
constexpr size_t kScratchBytes = kScrWork + kWorkBytes;
static_assert(kScrWork % 256 == 0 && kPartBytes % 256 == 0, "aligned sections");

void odometry_impl(void* ctx) {
    OdoCall& c = *static_cast<OdoCall*>(ctx);
    mp_filter f = c.f;
    if (!f || !c.p || !c.dT_out) mp_throw(MP_E_ARG, "null filter, parameters or output");
    const mp_odometry_params& P = *c.p;
    if (P.iterations < 0 || P.iterations > 1000 || !(P.d_max > 0.0f) || !std::isfinite(P.d_max) ||
        !(P.lambda_rel >= 0.0f) || !(P.lambda_abs >= 0.0f) || !(P.cov_scale > 0.0f) || !std::isfinite(P.cov_scale))
        mp_throw(MP_E_ARG, "iterations 0..1000, d_max > 0, damping >= 0 and cov_scale > 0 expected");
    if (f->scan_n <= 0 || f->prev_n <= 0)
        mp_throw(MP_E_STATE, "odometry needs two non-empty scans (mp_scan_upload twice)");
    double init[7] = {1, 0, 0, 0, 0, 0, 0};
    if (c.init) {
        for (int k = 0; k < 7; ++k) init[k] = c.init[k];
        double nq = 0.0;
        for (int k = 0; k < 4; ++k) nq += init[k] * init[k];
        for (int k = 0; k < 7; ++k)
            if (!std::isfinite(init[k])) mp_throw(MP_E_ARG, "non-finite initial dT");
        if (!(nq > 1e-12)) mp_throw(MP_E_ARG, "zero quaternion in the initial dT");
        for (int k = 0; k < 4; ++k) init[k] /= std::sqrt(nq);
    }
    hipStream_t s = c.s;
    const int ns = f->scan_n, nt = f->prev_n;
    // at most kOParts workgroups, each a run of consecutive points of the walk order
    const int rounds = std::max(1, (ns + kOSlots * kOParts - 1) / (kOSlots * kOParts));
    const int nparts = (ns + kOSlots * rounds - 1) / (kOSlots * rounds);
    int32_t* nn = nullptr;
    char* work = nullptr;
    if (c.scratch) {
        // the caller's fixed work area: no allocation
        if ((size_t)ns > kNoAllocScan)
            mp_throw(MP_E_ARG, "mp_odometry_noalloc: current scan of %d points exceeds its limit of %d", ns,
                     (int)kNoAllocScan);
        nn = reinterpret_cast<int32_t*>(c.scratch);
        work = c.scratch + kScrWork;
    } else {
        f->odo_nn.ensure(sizeof(int32_t) * (size_t)ns);
        f->odo_work.ensure(kWorkBytes);
        nn = f->odo_nn.as<int32_t>();
        work = f->odo_work.as<char>();
    }
    double* part[2] = {reinterpret_cast<double*>(work), reinterpret_cast<double*>(work + kPartBytes)};
    double* pose = reinterpret_cast<double*>(work + 2 * kPartBytes);
    double* out = pose + 16;
    const ScanIndex S = mp_scan_index(f->scan_idx, ns);
    OdoArgs A;
    A.T = mp_scan_index(f->prev_idx, nt);
    A.trec = f->prev_orig.as<float4>();
    A.swalk = (f->idx_own ? f->scan_own : f->scan).as<float4>();
    A.spts = S.pts;
    A.nn = nn;
    for (int k = 0; k < 7; ++k) A.init[k] = init[k];
    A.lam_rel = P.lambda_rel;
    A.lam_abs = P.lambda_abs;
    A.ns = ns;
    A.nparts = nparts;
    A.rounds = rounds;
    A.dmax2 = P.d_max * P.d_max;
    for (int it = 0; it <= P.iterations; ++it) {
        A.first = it == 0 ? 1 : 0;
        A.part_in = part[(it + 1) & 1];
        A.part_out = part[it & 1];
        A.pose_in = pose + 8 * ((it + 1) & 1);
        A.pose_out = pose + 8 * (it & 1);
        if (it < 2) k_odo_iter<true><<<(unsigned)nparts, kOThreads, 0, s>>>(A);
        else k_odo_iter<false><<<(unsigned)nparts, kOThreads, 0, s>>>(A);
        MP_CHECK_LAUNCH();
    }
    k_odo_final<<<1, kOThreads, 0, s>>>(part[P.iterations & 1], nparts, pose + 8 * (P.iterations & 1), P.cov_scale,
                                        out);
    MP_CHECK_LAUNCH();
    double h_state[kOutDoubles];
    MP_HIP(hipMemcpyAsync(h_state, out, sizeof(h_state), hipMemcpyDeviceToHost, s));
    MP_HIP(hipStreamSynchronize(s));
    const double* ho = h_state + 8;
    for (int k = 0; k < 7; ++k) c.dT_out[k] = (float)h_state[k];
    if (c.cov_out)
        for (int k = 0; k < 36; ++k) c.cov_out[k] = (float)ho[29 + k];
    if (c.res) {
        std::memset(c.res, 0, sizeof(*c.res));
        for (int k = 0; k < 21; ++k) c.res->H[k] = ho[k];
        for (int k = 0; k < 6; ++k) c.res->b[k] = ho[21 + k];
        c.res->cost = ho[27];
        c.res->inliers = (int32_t)ho[28];
        c.res->iterations = P.iterations;
        c.res->cov_ok = ho[65] != 0.0 ? 1 : 0;
        for (int k = 0; k < 7; ++k) c.res->dT64[k] = h_state[k];
    }
    f->last_stream = s;
}
}  // namespace

extern "C" mp_status mp_odometry(mp_filter f, const mp_odometry_params* params, const float init_dT[7], float dT_out[7],
                                 float cov_out[36], mp_odometry_result* result, void* stream) {
    OdoCall c{f, params, init_dT, dT_out, cov_out, result, static_cast<hipStream_t>(stream), nullptr};
    return mp_guarded_call("mp_odometry", odometry_impl, &c);
}

// Work area of mp_odometry_noalloc (0.18 MB): one copy per device, held until
// the process ends.  Host code never uses this name as an address: the device
// address comes from hipGetSymbolAddress, once per device.
static __device__ __align__(256) char scratch[kScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
char* g_scratch_ptr[kMaxDevices] = {};

// the device address of `scratch` on the current device (looked up on the
// first call there)
char* scratch_on_current_device() {
    int dev = -1;
    MP_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) mp_throw(MP_E_UNSUPPORTED, "device ordinal %d beyond %d", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        MP_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) mp_throw(MP_E_HIP, "hipGetSymbolAddress returned a null work area");
        g_scratch_ptr[dev] = static_cast<char*>(p);
    }
    return g_scratch_ptr[dev];
}

void odometry_noalloc_impl(void* ctx) {
    OdoCall& c = *static_cast<OdoCall*>(ctx);
    c.scratch = scratch_on_current_device();
    odometry_impl(ctx);
}
}  // namespace

extern "C" mp_status mp_odometry_noalloc(mp_filter f, const mp_odometry_params* params, const float init_dT[7],
                                         float dT_out[7], float cov_out[36], mp_odometry_result* result,
                                         void* stream) {
    OdoCall c{f, params, init_dT, dT_out, cov_out, result, static_cast<hipStream_t>(stream), nullptr};
    return mp_guarded_call("mp_odometry_noalloc", odometry_noalloc_impl, &c);
}
