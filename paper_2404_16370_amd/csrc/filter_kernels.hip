// filter_kernels.hip -- prediction (Eq. 1), SVGD update (Eq. 5-8),
// posterior propagation on the neighbour graph (Eq. 11) and initialisation.
#include <hip/hip_runtime.h>

#include <cmath>

#include "mp_det.hpp"
#include "mp_internal.hpp"
#include "mp_lsh.hpp"
#include "mp_many.hpp"

namespace {

inline unsigned nblk(int64_t n, int b = 256) { return (unsigned)((n + b - 1) / b); }

// SE(3) exponential of [omega; v] as (unit quaternion, translation), FP32.
//   q = (cos(th/2), sin(th/2)/th omega),  t = V v,
//   V = I + A [w]x + B [w]x^2, A = (1 - cos th)/th^2 = (sin(th/2)/(th/2))^2 / 2,
//   B = (th - sin th)/th^3 (series below th = 0.5).
__device__ inline void se3_exp(const float xi[6], mpdet::quat& q, float3& t) {
    const float wx = xi[0], wy = xi[1], wz = xi[2];
    const float th2 = wx * wx + wy * wy + wz * wz;
    const float th = sqrtf(th2);
    float hs, hc, A, B;
    if (th < 1e-4f) {
        hs = 0.5f - th2 * (1.0f / 48.0f);
        hc = 1.0f - th2 * 0.125f;
        A = 0.5f - th2 * (1.0f / 24.0f);
        B = 1.0f / 6.0f - th2 * (1.0f / 120.0f);
    } else {
        float sh, ch;
        sincosf(0.5f * th, &sh, &ch);
        hs = sh / th;
        hc = ch;
        const float sinc_half = sh / (0.5f * th);
        A = 0.5f * sinc_half * sinc_half;
        if (th < 0.5f) {
            B = 1.0f / 6.0f + th2 * (-1.0f / 120.0f + th2 * (1.0f / 5040.0f - th2 * (1.0f / 362880.0f)));
        } else {
            B = (th - sinf(th)) / (th2 * th);
        }
    }
    q = mpdet::quat{hc, hs * wx, hs * wy, hs * wz};
    const float vx = xi[3], vy = xi[4], vz = xi[5];
    const float c1x = wy * vz - wz * vy, c1y = wz * vx - wx * vz, c1z = wx * vy - wy * vx;
    const float c2x = wy * c1z - wz * c1y, c2y = wz * c1x - wx * c1z, c2z = wx * c1y - wy * c1x;
    t = make_float3(vx + A * c1x + B * c2x, vy + A * c1y + B * c2y, vz + A * c1z + B * c2z);
}

// (q, t) (x) (dq, dt) = (q dq, t + R(q) dt), quaternion renormalised
__device__ inline void compose(mpdet::quat& q, float3& t, const mpdet::quat dq, const float3 dt) {
    const mpdet::mat3 R = mpdet::qmat(q);
    t.x += R.m[0] * dt.x + R.m[1] * dt.y + R.m[2] * dt.z;
    t.y += R.m[3] * dt.x + R.m[4] * dt.y + R.m[5] * dt.z;
    t.z += R.m[6] * dt.x + R.m[7] * dt.y + R.m[8] * dt.z;
    mpdet::quat r = mpdet::qmul(q, dq);
    const float inv = rsqrtf(r.w * r.w + r.x * r.x + r.y * r.y + r.z * r.z);
    q = mpdet::quat{r.w * inv, r.x * inv, r.y * inv, r.z * inv};
}

__device__ inline void load_pose(const float4* P, int i, mpdet::quat& q, float3& t) {
    const float4 a = P[2 * i], b = P[2 * i + 1];
    q = mpdet::quat{a.x, a.y, a.z, a.w};
    t = make_float3(b.x, b.y, b.z);
}

__device__ inline void store_pose(float4* P, int i, const mpdet::quat q, const float3 t) {
    P[2 * i] = make_float4(q.w, q.x, q.y, q.z);
    P[2 * i + 1] = make_float4(t.x, t.y, t.z, 0.0f);
}

// ------------------------------------------------------------ SVGD
struct SvgdArgs {
    const float4* __restrict__ pin;
    float4* __restrict__ pout;
    const float4* __restrict__ psi;
    const int32_t* __restrict__ nbr;
    const float* __restrict__ kval;
    int32_t n, K;
    float sr, st;
    uint64_t* stamp;   // stage clock, or null
};

__device__ inline float3 cross3(const float3 a, const float3 b) {
    return float3{a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
__device__ inline float3 axpy3(float s, const float3 x, const float3 y) {
    return float3{s * x.x + y.x, s * x.y + y.y, s * x.z + y.z};
}

// J_r^-1(d)^T a for d = [om; rho], a = [aw; ar] (tangent order rotation
// first).  With M = I + 1/2 om^ + beta om^2 (the SO(3) inverse right
// Jacobian; beta as in the SE(3) logarithm) and Q(rho, om) the off-diagonal
// block of the SE(3) left Jacobian (Barfoot and Furgale, IEEE T-RO 2014):
//   J_r^-1(d) = [[M, 0], [-M Q(-rho, -om) M, M]],  Q(-rho, -om)^T = Q(rho, om),
// so that  v_r = M^T ar,  v_w = M^T (aw - Q(rho, om) v_r),
// M^T x = x - 1/2 om x x + beta om x (om x x).
__device__ inline void jr_inv_t(const float3 om, const float3 rho, float beta, const float3 aw, const float3 ar,
                                float3& vw, float3& vr) {
    auto mt = [&](const float3 x) {
        const float3 c1 = cross3(om, x);
        const float3 c2 = cross3(om, c1);
        return float3{(x.x - 0.5f * c1.x) + beta * c2.x, (x.y - 0.5f * c1.y) + beta * c2.y,
                      (x.z - 0.5f * c1.z) + beta * c2.z};
    };
    vr = mt(ar);
    const float th2 = (om.x * om.x + om.y * om.y) + om.z * om.z;
    float c1, c2, c3;   // (th - sin th)/th^3, (th^2 + 2 cos th - 2)/(2 th^4), (2 th - 3 sin th + th cos th)/(2 th^5)
    if (th2 < 1.0f) {   // Taylor series (cancellation in the closed forms below th = 1)
        c1 = fmaf(fmaf(fmaf(-1.0f / 362880.0f, th2, 1.0f / 5040.0f), th2, -1.0f / 120.0f), th2, 1.0f / 6.0f);
        c2 = fmaf(fmaf(fmaf(-1.0f / 3628800.0f, th2, 1.0f / 40320.0f), th2, -1.0f / 720.0f), th2, 1.0f / 24.0f);
        c3 = fmaf(fmaf(fmaf(-1.0f / 9979200.0f, th2, 1.0f / 120960.0f), th2, -1.0f / 2520.0f), th2, 1.0f / 120.0f);
    } else {
        const float th = sqrtf(th2);
        float sn, cs;
        sincosf(th, &sn, &cs);
        const float th4 = th2 * th2;
        c1 = (th - sn) / (th2 * th);
        c2 = (th2 + 2.0f * cs - 2.0f) / (2.0f * th4);
        c3 = (2.0f * th - 3.0f * sn + th * cs) / (2.0f * th4 * th);
    }
    // Q(rho, om) x = 1/2 rho^x + c1 (om^rho^ + rho^om^ + om^rho^om^) x
    //   + c2 (om^om^rho^ + rho^om^om^ - 3 om^rho^om^) x + c3 (om^rho^om^om^ + om^om^rho^om^) x
    const float3 b0 = cross3(rho, vr);
    const float3 a1 = cross3(om, vr);
    const float3 a2 = cross3(om, a1);
    const float3 b1 = cross3(rho, a1);
    const float3 b2 = cross3(rho, a2);
    const float3 wb0 = cross3(om, b0);
    const float3 wb1 = cross3(om, b1);
    const float3 wwb0 = cross3(om, wb0);
    const float3 wb2 = cross3(om, b2);
    const float3 wwb1 = cross3(om, wb1);
    float3 y;
    y.x = 0.5f * b0.x + c1 * (wb0.x + b1.x + wb1.x) + c2 * (wwb0.x + b2.x - 3.0f * wb1.x) + c3 * (wb2.x + wwb1.x);
    y.y = 0.5f * b0.y + c1 * (wb0.y + b1.y + wb1.y) + c2 * (wwb0.y + b2.y - 3.0f * wb1.y) + c3 * (wb2.y + wwb1.y);
    y.z = 0.5f * b0.z + c1 * (wb0.z + b1.z + wb1.z) + c2 * (wwb0.z + b2.z - 3.0f * wb1.z) + c3 * (wb2.z + wwb1.z);
    vw = mt(float3{aw.x - y.x, aw.y - y.y, aw.z - y.z});
}

// phi_i = sum_j v_ij / sum_j k_ij over the list of i, d_ij = log(T_i^-1 T_j),
// v_ij = k_ij psi_j + g_ij with the kernel gradient
//   EXACT = false   g = -2 k W d
//   EXACT = true    g = -2 k J_r^-1(d)^T W d
// and, with TRANSPORT, v_ij carried to T_i's tangent by Ad_{T_i^-1 T_j}:
//   [R v_w; t x (R v_w) + R v_r] with (R, t) = T_i^-1 T_j.
// T_i <- T_i exp(phi_i) (Jacobi: all j at pre-update poses).
// v_ij of one neighbour
template <bool EXACT, bool TRANSPORT>
__device__ __forceinline__ void svgd_term(const SvgdArgs& A, const mpdet::quat qi, const float3 ti, int j, float k,
                                          float v[6]) {
    mpdet::quat qj;
    float3 tj;
    load_pose(A.pin, j, qj, tj);
    float3 om, rho, tr;
    mpdet::quat qr;
    float beta;
    mpdet::se3_between_ex(qi, ti, qj, tj, om, rho, qr, tr, beta);
    const float4 p0 = A.psi[2 * j], p1 = A.psi[2 * j + 1];
    if (!EXACT && !TRANSPORT) {
        const float k2r = 2.0f * k * A.sr, k2t = 2.0f * k * A.st;
        v[0] = k * p0.x - k2r * om.x;
        v[1] = k * p0.y - k2r * om.y;
        v[2] = k * p0.z - k2r * om.z;
        v[3] = k * p0.w - k2t * rho.x;
        v[4] = k * p1.x - k2t * rho.y;
        v[5] = k * p1.y - k2t * rho.z;
    } else {
        float3 gw = float3{A.sr * om.x, A.sr * om.y, A.sr * om.z};
        float3 gr = float3{A.st * rho.x, A.st * rho.y, A.st * rho.z};
        if (EXACT) jr_inv_t(om, rho, beta, gw, gr, gw, gr);
        const float m2k = -2.0f * k;
        float3 vw = axpy3(m2k, gw, float3{k * p0.x, k * p0.y, k * p0.z});
        float3 vr = axpy3(m2k, gr, float3{k * p0.w, k * p1.x, k * p1.y});
        if (TRANSPORT) {
            const mpdet::mat3 R = mpdet::qmat(qr);
            const float3 rw = float3{R.m[0] * vw.x + R.m[1] * vw.y + R.m[2] * vw.z,
                                     R.m[3] * vw.x + R.m[4] * vw.y + R.m[5] * vw.z,
                                     R.m[6] * vw.x + R.m[7] * vw.y + R.m[8] * vw.z};
            const float3 rr = float3{R.m[0] * vr.x + R.m[1] * vr.y + R.m[2] * vr.z,
                                     R.m[3] * vr.x + R.m[4] * vr.y + R.m[5] * vr.z,
                                     R.m[6] * vr.x + R.m[7] * vr.y + R.m[8] * vr.z};
            const float3 tx = cross3(tr, rw);
            vw = rw;
            vr = float3{tx.x + rr.x, tx.y + rr.y, tx.z + rr.z};
        }
        v[0] = vw.x;
        v[1] = vw.y;
        v[2] = vw.z;
        v[3] = vr.x;
        v[4] = vr.y;
        v[5] = vr.z;
    }
}

// T_i exp(num / den), into qi, ti
__device__ __forceinline__ void svgd_move(const SvgdArgs& A, int i, mpdet::quat& qi, float3& ti, const float num[6],
                                          float den) {
    float phi[6];
    const float inv = den > 0.0f ? 1.0f / den : 0.0f;
    for (int m = 0; m < 6; ++m) phi[m] = num[m] * inv;
    mpdet::quat dq;
    float3 dt;
    se3_exp(phi, dq, dt);
    compose(qi, ti, dq, dt);
    store_pose(A.pout, i, qi, ti);
}

// 16 lanes per particle: lane l forms the terms of neighbours l and l + 16,
// then lane m < 7 adds component m (the sixth: k) over the list in list order.
// What bounds it: the gathers of the neighbours' poses and psi; with one lane
// per particle they follow one another.  From kSvMax particles on one lane each
// fills the chip, and leaves out the lists' empty places.  One lane / 16 lanes,
// K = 16, converged and spread (whose lists are nearly empty): 32,768 particles
// 27 / 11 us and 11 / 7, 65,536 29 / 20 and 12 / 12, 131,072 42 / 41 and 14 / 22,
// 1,048,576 506 / 455 and 60 / 146.
constexpr int kSvLanes = 16;
constexpr int kSvMax = 98304;

// L.codes: leave the codes of the next iteration's buckets as well (a launch
// less for each: ten iterations of 4096 particles 821 -> 794 us a frame)
template <bool EXACT, bool TRANSPORT>
__device__ __forceinline__ void svgd_rows(const SvgdArgs& A, LshArgs L, int block) {
    __shared__ float term[256 / kSvLanes][7][33];
    __shared__ float sum[256 / kSvLanes][8];
    __shared__ float sL[8];
    if (L.dyn) L.frame = L.dyn->frame;
    if (L.codes && threadIdx.x == 255) lsh_draw(L, sL, block == 0);
    const int gl = threadIdx.x % kSvLanes, g = threadIdx.x / kSvLanes;
    const int i0 = block * (256 / kSvLanes) + g;
    const int i = min(i0, A.n - 1);
    mpdet::quat qi;
    float3 ti;
    load_pose(A.pin, i, qi, ti);
    for (int a = gl; a < A.K; a += kSvLanes) {
        const int j = A.nbr[(size_t)a * A.n + i];
        float v[6] = {0, 0, 0, 0, 0, 0}, k = 0.0f;   // (no neighbour: adding zero changes no sum)
        if (j >= 0 && j < A.n) {
            k = A.kval[(size_t)a * A.n + i];
            svgd_term<EXACT, TRANSPORT>(A, qi, ti, j, k, v);
        }
        for (int m = 0; m < 6; ++m) term[g][m][a] = v[m];
        term[g][6][a] = k;
    }
    __syncthreads();
    if (gl < 7) {
        float s = 0.0f;
        for (int a = 0; a < A.K; ++a) s += term[g][gl][a];
        sum[g][gl] = s;
    }
    __syncthreads();
    // one lane per particle again
    if (threadIdx.x >= 256 / kSvLanes) return;
    const int p = block * (256 / kSvLanes) + threadIdx.x;
    if (p >= A.n) return;
    load_pose(A.pin, p, qi, ti);
    float num[6];
    for (int m = 0; m < 6; ++m) num[m] = sum[threadIdx.x][m];
    svgd_move(A, p, qi, ti, num, sum[threadIdx.x][6]);
    if (L.codes)
        lsh_code(L, sL, p, make_float4(qi.w, qi.x, qi.y, qi.z), make_float4(ti.x, ti.y, ti.z, 0.0f));
}

// one lane per particle
template <bool EXACT, bool TRANSPORT>
__device__ __forceinline__ void svgd_lanes(const SvgdArgs& A, LshArgs L, int block) {
    __shared__ float sL[8];
    if (L.dyn) L.frame = L.dyn->frame;
    if (L.codes && threadIdx.x == 255) lsh_draw(L, sL, block == 0);
    const int i = block * 256 + threadIdx.x;
    mpdet::quat qi;
    float3 ti;
    if (i < A.n) {
        load_pose(A.pin, i, qi, ti);
        float num[6] = {0, 0, 0, 0, 0, 0};
        float den = 0.0f;
        for (int a = 0; a < A.K; ++a) {
            const int j = A.nbr[(size_t)a * A.n + i];
            if (j < 0 || j >= A.n) continue;
            const float k = A.kval[(size_t)a * A.n + i];
            float v[6];
            svgd_term<EXACT, TRANSPORT>(A, qi, ti, j, k, v);
            for (int m = 0; m < 6; ++m) num[m] += v[m];
            den += k;
        }
        svgd_move(A, i, qi, ti, num, den);
    }
    if (!L.codes) return;   // (uniform)
    __syncthreads();
    if (i < A.n)
        lsh_code(L, sL, i, make_float4(qi.w, qi.x, qi.y, qi.z), make_float4(ti.x, ti.y, ti.z, 0.0f));
}

template <bool EXACT, bool TRANSPORT, bool ROWS>
__global__ __launch_bounds__(256) void k_svgd(SvgdArgs A, LshArgs L) {
    mp_write_stamp(A.stamp);
    if (ROWS) svgd_rows<EXACT, TRANSPORT>(A, L, blockIdx.x);
    else svgd_lanes<EXACT, TRANSPORT>(A, L, blockIdx.x);
}

struct SvgdLsh {
    SvgdArgs A;
    LshArgs L;
};

template <bool EXACT, bool TRANSPORT, bool ROWS>
__global__ __launch_bounds__(256) void k_svgd_many(Many<SvgdLsh> M) {
    int block;
    const SvgdLsh q = many_args(M, block);
    if (ROWS) svgd_rows<EXACT, TRANSPORT>(q.A, q.L, block);
    else svgd_lanes<EXACT, TRANSPORT>(q.A, q.L, block);
}

// ------------------------------------------------------------ prediction
struct PredArgs {
    float4* __restrict__ poses;
    int32_t n;
    uint32_t frame;
    uint64_t seed;
    float dq[4], dt[3];
    float L[21];  // lower-triangular Cholesky factor of the noise covariance, row-major packed
    int32_t noise;
    uint32_t purpose;                 // generator purpose of z (prediction, or Gaussian initialisation)
    const StepDyn* __restrict__ dyn;  // captured step: frame, increment and noise from here
    uint64_t* stamp;                  // stage clock, or null
    int32_t* flags;                   // the step's counters to clear, or null
};

__global__ __launch_bounds__(256) void k_predict(PredArgs A) {
    mp_write_stamp(A.stamp);
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (A.flags && i < 4) A.flags[i] = 0;
    if (i >= A.n) return;
    if (A.dyn) {
        if (!A.dyn->do_pred) return;
        A.frame = A.dyn->frame;
        A.noise = A.dyn->noise;
        for (int k = 0; k < 4; ++k) A.dq[k] = A.dyn->dq[k];
        for (int k = 0; k < 3; ++k) A.dt[k] = A.dyn->dt[k];
        for (int k = 0; k < 21; ++k) A.L[k] = A.dyn->L[k];
    }
    mpdet::quat q;
    float3 t;
    load_pose(A.poses, i, q, t);
    compose(q, t, mpdet::quat{A.dq[0], A.dq[1], A.dq[2], A.dq[3]}, make_float3(A.dt[0], A.dt[1], A.dt[2]));
    if (A.noise) {
        float z[6];
        mpdet::gauss6(A.seed, (uint32_t)i, A.frame, 0u, A.purpose, z);
        float d[6];
        int p = 0;
        for (int r = 0; r < 6; ++r) {
            float s = 0.0f;
            for (int c = 0; c <= r; ++c) s += A.L[p++] * z[c];
            d[r] = s;
        }
        mpdet::quat eq;
        float3 et;
        se3_exp(d, eq, et);
        compose(q, t, eq, et);
    }
    store_pose(A.poses, i, q, t);
}

// ------------------------------------------------------------ initialisation
struct InitArgs {
    float4* __restrict__ poses;
    int32_t n;
    uint64_t seed;
    float lo[3], hi[3];
};

__global__ __launch_bounds__(256) void k_init_uniform(InitArgs A) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= A.n) return;
    mpdet::quat q;
    float3 t;
    mpdet::random_pose(A.seed, (uint32_t)i, 0u, 0u, mpdet::PURPOSE_INIT, A.lo, A.hi, q, t);
    store_pose(A.poses, i, q, t);
}

// ------------------------------------------------------------ posterior
// Deterministic two-level reductions: per-block partials, then one block.  What
// bounds it is the launches, 3 to 5 us each: up to kRB partials are reduced by
// every block of the next kernel (one load a thread), the last round leaves the
// partials of its sums, and small filters take k_post_small.  Ten rounds, 65,536
// particles x 16 99 -> 71 us, 20,011 x 16 90 -> 63 us, 4097 x 8 71 -> 51 us;
// 1,048,576 x 16 961 -> 934 us converged, 292 -> 259 spread.
constexpr int kRB = 256;

__device__ inline double block_max(double v) {
    __shared__ double sh[kRB];
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int s = kRB / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) sh[threadIdx.x] = fmax(sh[threadIdx.x], sh[threadIdx.x + s]);
        __syncthreads();
    }
    const double r = sh[0];
    __syncthreads();
    return r;
}

__device__ inline double block_sum(double v) {
    __shared__ double sh[kRB];
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int s = kRB / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) sh[threadIdx.x] = sh[threadIdx.x] + sh[threadIdx.x + s];
        __syncthreads();
    }
    const double r = sh[0];
    __syncthreads();
    return r;
}

// (value, index) max, ties to the smaller index
__device__ inline void block_argmax(double& v, int& idx) {
    __shared__ double sv[kRB];
    __shared__ int si[kRB];
    sv[threadIdx.x] = v;
    si[threadIdx.x] = idx;
    __syncthreads();
    for (int s = kRB / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            const double a = sv[threadIdx.x], b = sv[threadIdx.x + s];
            const int ia = si[threadIdx.x], ib = si[threadIdx.x + s];
            if (b > a || (b == a && ib < ia)) {
                sv[threadIdx.x] = b;
                si[threadIdx.x] = ib;
            }
        }
        __syncthreads();
    }
    v = sv[0];
    idx = si[0];
    __syncthreads();
}

// stepinfo layout (doubles): 0 max l, 1 sum exp, 2 log evidence, 3 z, 4 map weight,
// 5 n_eff, 6 max loglik, 7 map index (as double)
struct PostArgs {
    const float* __restrict__ prior;
    const float4* __restrict__ psi;
    double* __restrict__ l;
    float* __restrict__ p0;
    float* __restrict__ p1;
    const int32_t* __restrict__ nbr;
    const float* __restrict__ kval;
    double* __restrict__ part;      // 3 x nblocks partials
    int* __restrict__ ipart;        // nblocks
    double* __restrict__ info;
    float* __restrict__ prior_out;
    int32_t n, K, nb;
    double inv_tau, floor_p;
    uint64_t* stamp;                // stage clock at the start, or null
    uint64_t* stamp_end;            // and at the end of the last launch, or null
};

__global__ __launch_bounds__(kRB) void k_post_logits(PostArgs A) {
    mp_write_stamp(A.stamp);
    const int i = blockIdx.x * kRB + threadIdx.x;
    double l = -INFINITY, ll = -INFINITY;
    if (i < A.n) {
        const double pr = fmax((double)A.prior[i], A.floor_p);
        ll = (double)A.psi[2 * i + 1].z;
        l = log(pr) + ll * A.inv_tau;
        A.l[i] = l;
    }
    const double m = block_max(l);
    const double mll = block_max(ll);
    if (threadIdx.x == 0) {
        A.part[blockIdx.x] = m;
        A.part[A.nb + blockIdx.x] = mll;
    }
}

// the partials' results, from every block of a launch (block 0 keeps them)
__device__ inline double post_max(const PostArgs& A) {
    double m = -INFINITY, mll = -INFINITY;
    for (int b = threadIdx.x; b < A.nb; b += kRB) {
        m = fmax(m, A.part[b]);
        mll = fmax(mll, A.part[A.nb + b]);
    }
    m = block_max(m);
    mll = block_max(mll);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        A.info[0] = m;
        A.info[6] = mll;
    }
    return m;
}

__device__ inline double post_sum(const PostArgs& A) {
    double s = 0.0;
    for (int b = threadIdx.x; b < A.nb; b += kRB) s += A.part[2 * A.nb + b];
    s = block_sum(s);
    const double ev = A.info[0] + log(s);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        A.info[1] = s;
        A.info[2] = ev;
    }
    return ev;
}

__device__ inline double post_z(const PostArgs& A) {
    double s = 0.0, v = -INFINITY;
    int idx = 0x7FFFFFFF;
    for (int b = threadIdx.x; b < A.nb; b += kRB) {
        s += A.part[b];
        const double vb = A.part[A.nb + b];
        const int ib = A.ipart[b];
        if (vb > v || (vb == v && ib < idx)) {
            v = vb;
            idx = ib;
        }
    }
    s = block_sum(s);
    block_argmax(v, idx);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        A.info[3] = s;
        A.info[4] = v / s;
        A.info[7] = (double)idx;
    }
    return s;
}

__global__ __launch_bounds__(kRB) void k_post_max_final(PostArgs A) { post_max(A); }
__global__ __launch_bounds__(kRB) void k_post_sum_final(PostArgs A) { post_sum(A); }
__global__ __launch_bounds__(kRB) void k_post_z_final(PostArgs A) { post_z(A); }

// WIDE: more partials than one block reads at once; a launch of its own reduced them
template <bool WIDE>
__global__ __launch_bounds__(kRB) void k_post_expsum(PostArgs A) {
    const int i = blockIdx.x * kRB + threadIdx.x;
    const double m = WIDE ? A.info[0] : post_max(A);
    const double e = (i < A.n) ? exp(A.l[i] - m) : 0.0;
    const double s = block_sum(e);
    if (threadIdx.x == 0) A.part[2 * A.nb + blockIdx.x] = s;   // the maxima are still being read
}

template <bool WIDE>
__global__ __launch_bounds__(kRB) void k_post_normalise(PostArgs A) {
    const int i = blockIdx.x * kRB + threadIdx.x;
    const double ev = WIDE ? A.info[2] : post_sum(A);
    if (i >= A.n) return;
    A.p0[i] = (float)exp(A.l[i] - ev);
}

// one Jacobi round of Eq. 11: p'_i = sum_j k_ij p_j / sum_j k_ij.  Eight
// neighbours' loads are in flight before the first is added.
__device__ inline float post_average(const PostArgs& A, const float* __restrict__ pin, int i) {
    constexpr int kU = 8;
    const size_t n = (size_t)A.n;
    float num = 0.0f, den = 0.0f;
    const float own = pin[i];
    for (int a0 = 0; a0 < A.K; a0 += kU) {
        int32_t j[kU];
        float k[kU], p[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            j[u] = A.nbr[(size_t)min(a0 + u, A.K - 1) * n + i];
            if (a0 + u >= A.K || j[u] >= A.n) j[u] = -1;
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {   // (an empty place costs no load)
            k[u] = 0.0f;
            p[u] = 0.0f;
            if (j[u] >= 0) {
                k[u] = A.kval[(size_t)(a0 + u) * n + i];
                p[u] = pin[j[u]];
            }
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            num = j[u] >= 0 ? num + k[u] * p[u] : num;
            den = j[u] >= 0 ? den + k[u] : den;
        }
    }
    return den > 0.0f ? num / den : own;
}

// sum and largest of the weights: this block's partials
__device__ inline void post_z_part(const PostArgs& A, float p, int i) {
    double v = -INFINITY;
    int idx = 0x7FFFFFFF;
    double s = 0.0;
    if (i < A.n) {
        v = (double)p;
        idx = i;
        s = v;
    }
    s = block_sum(s);
    block_argmax(v, idx);
    if (threadIdx.x == 0) {
        A.part[blockIdx.x] = s;
        A.part[A.nb + blockIdx.x] = v;
        A.ipart[blockIdx.x] = idx;
    }
}

template <bool LAST>
__global__ __launch_bounds__(kRB) void k_post_round(PostArgs A, const float* __restrict__ pin,
                                                    float* __restrict__ pout) {
    const int i = blockIdx.x * kRB + threadIdx.x;
    float p = 0.0f;
    if (i < A.n) pout[i] = p = post_average(A, pin, i);
    if (LAST) post_z_part(A, p, i);
}

__global__ __launch_bounds__(kRB) void k_post_z(PostArgs A, const float* __restrict__ p) {   // without a round
    const int i = blockIdx.x * kRB + threadIdx.x;
    post_z_part(A, i < A.n ? p[i] : 0.0f, i);
}

template <bool WIDE>
__global__ __launch_bounds__(kRB) void k_post_store(PostArgs A, const float* __restrict__ p) {
    const int i = blockIdx.x * kRB + threadIdx.x;
    const double z = WIDE ? A.info[3] : post_z(A);
    double q = 0.0;
    if (i < A.n) {
        q = (double)p[i] / z;
        A.prior_out[i] = (float)q;
    }
    const double s = block_sum(q * q);
    if (threadIdx.x == 0) A.part[2 * A.nb + blockIdx.x] = s;
}

__global__ __launch_bounds__(kRB) void k_post_neff_final(PostArgs A) {
    double s = 0.0;
    for (int b = threadIdx.x; b < A.nb; b += kRB) s += A.part[2 * A.nb + b];
    s = block_sum(s);
    if (threadIdx.x == 0) A.info[5] = 1.0 / s;
    mp_write_stamp(A.stamp_end);
}

// The whole posterior in one workgroup, for filters whose lists fit its
// registers: T threads, particle r * T + thread its r-th, kPostSlots /
// R list slots each.  Wave w reduces particles [256 w, 256 (w + 1)) and the
// results are reduced as above, in the same trees, so it gives the same bits.
// What bounds it: one CU's LDS gathers and FP64 exp and log.  Ten rounds, 256
// particles x 8 54 -> 14 us (19 with 1024 threads, which wait longer at the
// barriers), 1000 x 16 80 -> 23 us, 4096 x 8 71 -> 37 us (49 in the launches
// above).  Lists kept in more registers would spill.
constexpr int kPT = 1024;
constexpr int kPostSlots = 32;

// wave w's tree over its 256 values of v (4 a lane) as block_sum adds them
__device__ inline double wave_sum(const double* v, int lane) {
    double x = (v[lane] + v[lane + 128]) + (v[lane + 64] + v[lane + 192]);
    for (int s = 32; s > 0; s >>= 1) x = x + __shfl_down(x, s);
    return __shfl(x, 0);
}

// sum over the blocks' partials
__device__ inline double parts_sum(const double* part, int nb, int lane) {
    double x = lane < nb ? part[lane] : 0.0;
    for (int s = kPT / kRB / 2 * 4; s > 0; s >>= 1) x = x + __shfl_down(x, s);
    return __shfl(x, 0);
}

__device__ inline void pick(double& v, int& idx, double b, int ib) {
    if (b > v || (b == v && ib < idx)) {
        v = b;
        idx = ib;
    }
}

template <int R, int T = kPT>
__global__ __launch_bounds__(T) void k_post_small(PostArgs A, int rounds) {
    constexpr int N = R * T, KC = kPostSlots / R, W = T / 64;
    __shared__ double sh[N];
    __shared__ float pb[2][N + 1];   // and a zero
    __shared__ double part[3][W];
    __shared__ int ipart[W];
    mp_write_stamp(A.stamp);
    if (threadIdx.x < 2) pb[threadIdx.x][N] = 0.0f;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int n = A.n;
    int32_t j[R][KC];
    float kv[R][KC];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int a = 0; a < KC; ++a) {
            const int i = r * T + tid;
            const bool in = a < A.K && i < n;
            const size_t at = in ? (size_t)a * n + i : 0;
            const int32_t x = A.nbr[at];
            const float k = A.kval[at];
            const bool valid = in && x >= 0 && x < n;
            kv[r][a] = valid ? k : 0.0f;   // an empty slot adds 0 * 0
            j[r][a] = valid ? x : N;
        }
    // logits and their maximum
    double m = -INFINITY, mll = -INFINITY;
#pragma unroll 1
    for (int i = tid; i < n; i += T) {
        const double pr = fmax((double)A.prior[i], A.floor_p);
        const double ll = (double)A.psi[2 * i + 1].z;
        const double l = log(pr) + ll * A.inv_tau;
        sh[i] = l;
        m = fmax(m, l);
        mll = fmax(mll, ll);
    }
    for (int s = 32; s > 0; s >>= 1) {
        m = fmax(m, __shfl_xor(m, s));
        mll = fmax(mll, __shfl_xor(mll, s));
    }
    if (lane == 0) {
        part[0][wave] = m;
        part[1][wave] = mll;
    }
    __syncthreads();
    m = lane < W ? part[0][lane] : -INFINITY;
    mll = lane < W ? part[1][lane] : -INFINITY;
    for (int s = 32; s > 0; s >>= 1) {
        m = fmax(m, __shfl_xor(m, s));
        mll = fmax(mll, __shfl_xor(mll, s));
    }
    // evidence
    double l[R];
#pragma unroll
    for (int r = 0; r < R; ++r) l[r] = sh[r * T + tid];   // own values: of no thread beyond n
    for (int r = 0; r < R; ++r) {
        const int i = r * T + tid;
        sh[i] = i < n ? exp(sh[i] - m) : 0.0;
    }
    __syncthreads();
    if (wave < A.nb) {
        const double s = wave_sum(sh + wave * kRB, lane);
        if (lane == 0) part[2][wave] = s;
    }
    __syncthreads();
    const double sum = parts_sum(part[2], A.nb, lane);
    const double ev = m + log(sum);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * T + tid;
        pb[0][i] = i < n ? (float)exp(l[r] - ev) : 0.0f;
        pb[1][i] = 0.0f;
    }
    // rounds
    int cur = 0;
    for (int it = 0; it < rounds; ++it, cur ^= 1) {
        __syncthreads();
        const float* pin = pb[cur];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = r * T + tid;
            float num = 0.0f, den = 0.0f;
#pragma unroll
            for (int a = 0; a < KC; ++a) {
                if (a < A.K) {
                    num = num + kv[r][a] * pin[j[r][a]];
                    den = den + kv[r][a];
                }
            }
            pb[cur ^ 1][i] = den > 0.0f ? num / den : pin[i];
        }
    }
    // sum and largest weight
    __syncthreads();
    const float* pf = pb[cur];
    if (wave < A.nb) {
        const int at = wave * kRB + lane;
        double x[4];
        for (int q = 0; q < 4; ++q) x[q] = at + 64 * q < n ? (double)pf[at + 64 * q] : 0.0;
        double s = (x[0] + x[2]) + (x[1] + x[3]);
        for (int q = 0; q < 4; ++q) x[q] = at + 64 * q < n ? x[q] : -INFINITY;
        int idx = at < n ? at : 0x7FFFFFFF, idx1 = at + 64 < n ? at + 64 : 0x7FFFFFFF;
        double v = x[0], v1 = x[1];
        pick(v, idx, x[2], at + 128 < n ? at + 128 : 0x7FFFFFFF);
        pick(v1, idx1, x[3], at + 192 < n ? at + 192 : 0x7FFFFFFF);
        pick(v, idx, v1, idx1);
        for (int d = 32; d > 0; d >>= 1) {
            s = s + __shfl_down(s, d);
            pick(v, idx, __shfl_down(v, d), __shfl_down(idx, d));
        }
        if (lane == 0) {
            part[0][wave] = s;
            part[1][wave] = v;
            ipart[wave] = idx;
        }
    }
    __syncthreads();
    const double z = parts_sum(part[0], A.nb, lane);
    double v = -INFINITY;
    int idx = 0x7FFFFFFF;
    if (lane < A.nb) pick(v, idx, part[1][lane], ipart[lane]);
    for (int d = 32; d > 0; d >>= 1) pick(v, idx, __shfl_down(v, d), __shfl_down(idx, d));
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * T + tid;
        double q = 0.0;
        if (i < n) {
            q = (double)pf[i] / z;
            A.prior_out[i] = (float)q;
            A.p0[i] = pb[0][i];
            A.p1[i] = pb[1][i];
        }
        sh[i] = q * q;
    }
    __syncthreads();
    if (wave < A.nb) {
        const double s = wave_sum(sh + wave * kRB, lane);
        if (lane == 0) part[2][wave] = s;
    }
    __syncthreads();
    const double q2 = parts_sum(part[2], A.nb, lane);
    if (tid == 0) {
        A.info[0] = m;
        A.info[1] = sum;
        A.info[2] = ev;
        A.info[3] = z;
        A.info[4] = v / z;
        A.info[5] = 1.0 / q2;
        A.info[6] = mll;
        A.info[7] = (double)idx;
    }
    mp_write_stamp(A.stamp_end);
}

// the end of a step whose last kernel does not stamp it
__global__ void k_stamp(uint64_t* p) { mp_write_stamp(p); }

}  // namespace

// (leaves the update's poses current)
static SvgdLsh svgd_args(mp_filter f, const LshArgs* next) {
    SvgdLsh q;
    SvgdArgs& A = q.A;
    A.pin = f->poses[f->cur].as<float4>();
    A.pout = f->poses[1 - f->cur].as<float4>();
    A.psi = f->psi.as<float4>();
    A.nbr = f->nbr.as<int32_t>();
    A.kval = f->kval.as<float>();
    A.n = f->n;
    A.K = f->K;
    A.sr = f->p.sigma_r;
    A.st = f->p.sigma_t;
    A.stamp = nullptr;
    if (next) {
        q.L = *next;
    } else {
        q.L.codes = nullptr;
        q.L.dyn = nullptr;
    }
    f->cur = 1 - f->cur;
    return q;
}

// variant: gradient, transport, lanes per particle
static int svgd_kind(mp_filter f) {
    return (f->p.svgd_grad == MP_SVGD_GRAD_EXACT ? 4 : 0) + (f->p.svgd_transport == MP_SVGD_TRANSPORT_ADJOINT ? 2 : 0) +
           (f->n <= kSvMax ? 1 : 0);
}

static unsigned svgd_blocks(mp_filter f) { return nblk(f->n, f->n <= kSvMax ? 256 / kSvLanes : 256); }

void mp_launch_svgd(mp_filter f, hipStream_t s, const LshArgs* next) {
    SvgdLsh q = svgd_args(f, next);
    q.A.stamp = mp_take_stamp(f);
    const unsigned grid = svgd_blocks(f);
    switch (svgd_kind(f)) {
        case 7: k_svgd<true, true, true><<<grid, 256, 0, s>>>(q.A, q.L); break;
        case 6: k_svgd<true, true, false><<<grid, 256, 0, s>>>(q.A, q.L); break;
        case 5: k_svgd<true, false, true><<<grid, 256, 0, s>>>(q.A, q.L); break;
        case 4: k_svgd<true, false, false><<<grid, 256, 0, s>>>(q.A, q.L); break;
        case 3: k_svgd<false, true, true><<<grid, 256, 0, s>>>(q.A, q.L); break;
        case 2: k_svgd<false, true, false><<<grid, 256, 0, s>>>(q.A, q.L); break;
        case 1: k_svgd<false, false, true><<<grid, 256, 0, s>>>(q.A, q.L); break;
        default: k_svgd<false, false, false><<<grid, 256, 0, s>>>(q.A, q.L);
    }
    MP_CHECK_LAUNCH();
}

void mp_many_svgd(const std::vector<mp_filter>& fs, int it, ManyTab& T, hipStream_t s) {
    for (int kind = 0; kind < 8; ++kind) {
        std::vector<SvgdLsh> a;
        std::vector<int32_t> blocks;
        for (mp_filter f : fs) {
            if (svgd_kind(f) != kind) continue;
            const bool more = it + 1 < f->p.svgd_iters;
            const LshArgs next = mp_lsh_args(f, (uint32_t)f->frame, (uint32_t)((it + 1) * std::max(1, f->p.lsh_tables)));
            a.push_back(svgd_args(f, more ? &next : nullptr));
            f->lsh_ahead = more;
            blocks.push_back((int32_t)svgd_blocks(f));
        }
        if (a.empty()) continue;
        unsigned grid;
        const Many<SvgdLsh> M = many_table(T, a, blocks, grid);
        switch (kind) {
            case 7: k_svgd_many<true, true, true><<<grid, 256, 0, s>>>(M); break;
            case 6: k_svgd_many<true, true, false><<<grid, 256, 0, s>>>(M); break;
            case 5: k_svgd_many<true, false, true><<<grid, 256, 0, s>>>(M); break;
            case 4: k_svgd_many<true, false, false><<<grid, 256, 0, s>>>(M); break;
            case 3: k_svgd_many<false, true, true><<<grid, 256, 0, s>>>(M); break;
            case 2: k_svgd_many<false, true, false><<<grid, 256, 0, s>>>(M); break;
            case 1: k_svgd_many<false, false, true><<<grid, 256, 0, s>>>(M); break;
            default: k_svgd_many<false, false, false><<<grid, 256, 0, s>>>(M);
        }
        MP_CHECK_LAUNCH();
    }
}

void mp_launch_predict(mp_filter f, const float dT[7], const float L[36], bool noise, hipStream_t s,
                       bool gauss_init) {
    PredArgs A;
    A.purpose = gauss_init ? mpdet::PURPOSE_INIT_GAUSS : mpdet::PURPOSE_PRED;
    A.poses = f->poses[f->cur].as<float4>();
    A.n = f->n;
    A.frame = (uint32_t)f->frame;
    A.seed = f->p.seed;
    for (int k = 0; k < 4; ++k) A.dq[k] = dT[k];
    for (int k = 0; k < 3; ++k) A.dt[k] = dT[4 + k];
    int p = 0;
    for (int r = 0; r < 6; ++r)
        for (int c = 0; c <= r; ++c) A.L[p++] = noise ? L[6 * r + c] : 0.0f;
    A.noise = noise ? 1 : 0;
    A.dyn = f->dyn;
    A.flags = mp_take_flags(f);
    A.stamp = mp_take_stamp(f);
    k_predict<<<nblk(f->n), 256, 0, s>>>(A);
    MP_CHECK_LAUNCH();
}

void mp_launch_init_uniform(mp_filter f, const float lo[3], const float hi[3], hipStream_t s) {
    InitArgs A;
    A.poses = f->poses[f->cur].as<float4>();
    A.n = f->n;
    A.seed = f->p.seed;
    for (int a = 0; a < 3; ++a) {
        A.lo[a] = lo[a];
        A.hi[a] = hi[a];
    }
    k_init_uniform<<<nblk(f->n), 256, 0, s>>>(A);
    MP_CHECK_LAUNCH();
}

size_t mp_post_scratch_bytes(mp_filter f) {
    // l (n doubles), partials (3 nb doubles), index partials (nb ints)
    const int nb = (int)nblk(f->n, kRB);
    return sizeof(double) * ((size_t)f->n + 3 * (size_t)nb) + sizeof(int) * (size_t)nb + 64;
}

__global__ void k_fill_u32(uint32_t* __restrict__ p, uint32_t v, size_t n) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

void mp_fill_u32(void* p, uint32_t v, size_t n, hipStream_t s) {
    if (n == 0) return;
    k_fill_u32<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(static_cast<uint32_t*>(p), v, n);
    MP_CHECK_LAUNCH();
}

__global__ void k_copy_f4(const float4* __restrict__ src, float4* __restrict__ dst, size_t n) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

void mp_copy_poses(mp_filter f, int from, int to, hipStream_t s) {
    const size_t n = 2 * (size_t)f->n;
    k_copy_f4<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(f->poses[from].as<float4>(), f->poses[to].as<float4>(), n);
    MP_CHECK_LAUNCH();
}

namespace {
struct QueryArgs {
    const float4* __restrict__ poses;
    const float* __restrict__ prior;
    const double* __restrict__ info;
    const int32_t* __restrict__ flags;
    QueryOut* out;     // host memory
    float* pout;       // m x 7, or null
    double* wout;      // m, or null
    int32_t n;
    int32_t i0, m;     // the particles that are handed out
};

// Packing and the finiteness check of what a query hands out, one thread per
// four bytes of a pose, so that the stores are whole runs (device memory, or
// the host's over the link).
__global__ __launch_bounds__(256) void k_query(QueryArgs A) {
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const float* P = reinterpret_cast<const float*>(A.poses);
    bool bad = false;
    if (A.pout && q < 7 * (int64_t)A.m) {
        const int64_t i = q / 7;
        const float v = P[8 * (A.i0 + i) + (q - 7 * i)];
        bad = !isfinite(v);
        A.pout[q] = v;
    }
    if (A.wout && q < A.m) {
        const float v = A.prior[A.i0 + q];
        bad = bad || !isfinite(v);
        A.wout[q] = (double)v;
    }
    if (bad) __hip_atomic_store(&A.out->bad, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (q == 0 && A.i0 == 0) {
        for (int k = 0; k < 8; ++k) A.out->info[k] = A.info[k];
        int idx = (int)A.info[7];
        if (idx < 0 || idx >= A.n) idx = 0;
        for (int k = 0; k < 8; ++k) A.out->pose[k] = P[8 * (int64_t)idx + k];
        A.out->index = idx;
        A.out->resolves = A.flags[0];
    }
}
}  // namespace

void mp_launch_query(mp_filter f, QueryOut* out, float* poses, double* weights, int32_t i0, int32_t m,
                     hipStream_t s) {
    QueryArgs A;
    A.poses = f->poses[f->cur].as<float4>();
    A.prior = f->prior.as<float>();
    A.info = f->stepinfo.as<double>();
    A.flags = f->flags.as<int32_t>();
    A.out = out;
    A.pout = poses;
    A.wout = weights;
    A.n = f->n;
    A.i0 = i0;
    A.m = m;
    const int64_t items = poses ? 7 * (int64_t)m : (weights ? (int64_t)m : 1);
    k_query<<<nblk(items), 256, 0, s>>>(A);
    MP_CHECK_LAUNCH();
}

void mp_launch_stamp(uint64_t* p, hipStream_t s) {
    k_stamp<<<1, 64, 0, s>>>(p);
    MP_CHECK_LAUNCH();
}

void mp_launch_posterior(mp_filter f, hipStream_t s, uint64_t* stamp_end) {
    const int n = f->n;
    const int nb = (int)nblk(n, kRB);
    f->red.ensure(mp_post_scratch_bytes(f));
    PostArgs A;
    A.prior = f->prior.as<float>();
    A.psi = f->psi.as<float4>();
    A.l = f->red.as<double>();
    A.part = A.l + n;
    A.ipart = reinterpret_cast<int*>(A.part + 3 * (size_t)nb);
    A.p0 = f->post0.as<float>();
    A.p1 = f->post1.as<float>();
    A.nbr = f->nbr.as<int32_t>();
    A.kval = f->kval.as<float>();
    A.info = f->stepinfo.as<double>();
    A.prior_out = f->prior.as<float>();
    A.n = n;
    A.K = f->K;
    A.nb = nb;
    A.inv_tau = 1.0 / (double)f->p.temperature;
    A.floor_p = (double)f->p.prior_floor;
    A.stamp = mp_take_stamp(f);
    A.stamp_end = stamp_end;
    const int rounds = f->p.post_iters;
    // one workgroup while a lane's list slots fit its registers
    const int slots = f->K * ((n + kPT - 1) / kPT);
    if (n <= kPT / 4 && slots <= kPostSlots) {
        k_post_small<1, kPT / 4><<<1, kPT / 4, 0, s>>>(A, rounds);
    } else if (n <= kPT && slots <= kPostSlots) {
        k_post_small<1><<<1, kPT, 0, s>>>(A, rounds);
    } else if (n <= 2 * kPT && slots <= kPostSlots) {
        k_post_small<2><<<1, kPT, 0, s>>>(A, rounds);
    } else if (n <= 4 * kPT && 4 * f->K <= kPostSlots) {
        k_post_small<4><<<1, kPT, 0, s>>>(A, rounds);
    } else {
        const bool wide = nb > kRB;
        k_post_logits<<<nb, kRB, 0, s>>>(A);
        if (wide) {
            k_post_max_final<<<1, kRB, 0, s>>>(A);
            k_post_expsum<true><<<nb, kRB, 0, s>>>(A);
            k_post_sum_final<<<1, kRB, 0, s>>>(A);
            k_post_normalise<true><<<nb, kRB, 0, s>>>(A);
        } else {
            k_post_expsum<false><<<nb, kRB, 0, s>>>(A);
            k_post_normalise<false><<<nb, kRB, 0, s>>>(A);
        }
        float* a = A.p0;
        float* b = A.p1;
        for (int r = 0; r < rounds; ++r) {
            if (r + 1 < rounds) k_post_round<false><<<nb, kRB, 0, s>>>(A, a, b);
            else k_post_round<true><<<nb, kRB, 0, s>>>(A, a, b);
            float* t = a;
            a = b;
            b = t;
        }
        if (rounds <= 0) k_post_z<<<nb, kRB, 0, s>>>(A, a);
        if (wide) {
            k_post_z_final<<<1, kRB, 0, s>>>(A);
            k_post_store<true><<<nb, kRB, 0, s>>>(A, a);
        } else {
            k_post_store<false><<<nb, kRB, 0, s>>>(A, a);
        }
        k_post_neff_final<<<1, kRB, 0, s>>>(A);
    }
    MP_CHECK_LAUNCH();
}
