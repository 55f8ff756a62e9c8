// scan.hip -- scan point Gaussians (Sec. III-C: every scan point is modelled
// as N(mu, Sigma), GICP after Segal et al. 2009).
//
// mu is the point itself.  Without caller covariances, Sigma is the
// GICP-normalised covariance I - (1-eps) n n^T of the point and its k nearest
// other scan points: k-NN by FP32 squared distance (fixed fma order, ties to
// the lower index; a spatial index skips what is too far, 16 lanes per point), FP64 mean and 1/(k+1)
// covariance summed self-first in neighbour order, FP64 cyclic Jacobi with a
// fixed operation order.  Fewer than 5 points give Sigma = I.
//
// Record layout consumed by the likelihood kernel (3 float4 per point):
//   (mu_x, mu_y, mu_z, S_xx), (S_xy, S_xz, S_yy, S_yz), (S_zz, 0, 0, 0)
#include <hip/hip_runtime.h>

#include "mp_internal.hpp"
#include "mp_scan_index.hpp"

namespace {

constexpr int kB = 256;   // 16 points per workgroup
constexpr int kKMax = 32;

// Cyclic Jacobi on a symmetric 3x3 (row-major) and the eigenvector of the
// smallest eigenvalue (lowest index on ties).  The rotation loop is unrolled
// so that every index into A and V is a constant and both stay in registers.
__device__ void jacobi_min_vec(double A[9], double nrm[3]) {
    double V[9] = {1, 0, 0, 0, 1, 0, 0, 0, 1};
    for (int sweep = 0; sweep < 60; ++sweep) {
        const double off = A[1] * A[1] + A[2] * A[2] + A[5] * A[5];
        const double dg = A[0] * A[0] + A[4] * A[4] + A[8] * A[8];
        if (off <= 1e-300 || off <= 1e-34 * dg) break;
#pragma unroll
        for (int pq = 0; pq < 3; ++pq) {
            const int p = pq == 2 ? 1 : 0;
            const int q = pq == 0 ? 1 : 2;
            const double apq = A[3 * p + q];
            if (apq == 0.0) continue;
            const double app = A[3 * p + p], aqq = A[3 * q + q];
            const double th = (aqq - app) / (2.0 * apq);
            const double t = (th >= 0 ? 1.0 : -1.0) / (fabs(th) + sqrt(th * th + 1.0));
            const double c = 1.0 / sqrt(t * t + 1.0);
            const double s = t * c;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const double x = A[3 * k + p], y = A[3 * k + q];
                A[3 * k + p] = c * x - s * y;
                A[3 * k + q] = s * x + c * y;
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const double x = A[3 * p + k], y = A[3 * q + k];
                A[3 * p + k] = c * x - s * y;
                A[3 * q + k] = s * x + c * y;
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const double x = V[3 * k + p], y = V[3 * k + q];
                V[3 * k + p] = c * x - s * y;
                V[3 * k + q] = s * x + c * y;
            }
        }
    }
    int m = 0;
    if (A[4] < A[0]) m = 1;
    if (A[8] < (m == 1 ? A[4] : A[0])) m = 2;
    nrm[0] = m == 0 ? V[0] : (m == 1 ? V[1] : V[2]);
    nrm[1] = m == 0 ? V[3] : (m == 1 ? V[4] : V[5]);
    nrm[2] = m == 0 ? V[6] : (m == 1 ? V[7] : V[8]);
}

// raises *p to the device clock at which the workgroup ends
__device__ __forceinline__ void stamp_last(uint64_t* p) {
    __syncthreads();
    if (threadIdx.x == 0) atomicMax((unsigned long long*)p, (unsigned long long)wall_clock64());
}

// ------------------------------------------------------------ spatial index of a scan
// The scan in the likelihood's walk order (Morton order of its cells) or one of
// its own (k_index_keys below), as (x, y, z, caller index) per point, with the
// bounding boxes of every block of 64 consecutive points and of every 16 blocks:
// the neighbour searches (here and in the odometry) skip a box when it lies
// farther away than what they already hold.  One workgroup per 1024 points, one
// wave per block.
constexpr int kIdxThreads = kScanBlock * kScanFan;

// minimum over the wave (every lane active): within rows of 16, then over the
// rows (an upload of 8192 points 73.1 us, 75.1 with shuffles over the wave)
__device__ __forceinline__ float wave_min(float v) {
    const int m = __float_as_int(mp_row_min(v));
    const auto row = [&](int r) { return __int_as_float(__builtin_amdgcn_readlane(m, 16 * r)); };
    return fminf(fminf(row(0), row(1)), fminf(row(2), row(3)));
}

__global__ __launch_bounds__(kIdxThreads) void k_scan_index(const float* __restrict__ xyz,
                                                            const int32_t* __restrict__ perm, int n, ScanIndex X,
                                                            const uint64_t* __restrict__ start,
                                                            uint64_t* __restrict__ stamps) {
    __shared__ float box[kScanFan][6];
    if (blockIdx.x == 0 && threadIdx.x == 0) {   // the upload stands: its clock values
        stamps[0] = *start;
        stamps[1] = 0;
    }
    const int w = blockIdx.x * kIdxThreads + threadIdx.x;
    float b[6];   // lower corner, negated upper corner: both are minima
#pragma unroll
    for (int a = 0; a < 6; ++a) b[a] = __builtin_inff();
    if (w < n) {
        const int j = perm[w];
        const float x = xyz[3 * j], y = xyz[3 * j + 1], z = xyz[3 * j + 2];
        X.pts[w] = make_float4(x, y, z, __int_as_float(j));
        b[0] = x; b[1] = y; b[2] = z;
        b[3] = -x; b[4] = -y; b[5] = -z;
    }
#pragma unroll
    for (int a = 0; a < 6; ++a) b[a] = wave_min(b[a]);
    const int v = threadIdx.x / kScanBlock;
    if (threadIdx.x % kScanBlock == 0) {
#pragma unroll
        for (int a = 0; a < 6; ++a) box[v][a] = b[a];
        const int blk = blockIdx.x * kScanFan + v;
        if (blk < X.blocks) {
            X.box[2 * blk] = make_float4(b[0], b[1], b[2], 0.0f);
            X.box[2 * blk + 1] = make_float4(-b[3], -b[4], -b[5], 0.0f);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int u = 1; u < kScanFan; ++u)
#pragma unroll
            for (int a = 0; a < 6; ++a) b[a] = fminf(b[a], box[u][a]);
        X.super[2 * blockIdx.x] = make_float4(b[0], b[1], b[2], 0.0f);
        X.super[2 * blockIdx.x + 1] = make_float4(-b[3], -b[4], -b[5], 0.0f);
    }
}

// k nearest other scan points of each point, 16 lanes per point.  The lanes
// test the boxes of the index 16 at a time, first those of 1024 points, then
// the 16 blocks of each that may hold a neighbour; of a block that passes,
// every lane takes four points.  The row's list is sorted across its lanes
// (lane l keeps the l-th and, for k > 16, the (16 + l)-th smallest (d2, j)): a
// candidate within the k-th distance is handed to all lanes, each of which
// keeps its own entry, the candidate or the entry of the lane before.  Then the
// FP64 Gaussian of the point and its neighbours, a lane per sum, and the
// eigen-solves of the workgroup's 16 points side by side in one wave.
//
// What bounds it: latency of the insertions and of the eigen-solve (some 30
// dependent FP64 divisions and roots).  300 points take 21 us, 8192 32 us and
// 65,536 110 us; with a list per lane, a merge, the boxes in index order and an
// eigen-solve per wave of four points it took 30, 54 and 220 us, and a search
// through all n points, staged in LDS, 290 us for 8192 and 4.6 ms for 65,536.
constexpr int kQLanes = 16;
static_assert(kScanFan == kQLanes, "one lane per block of a box of 1024 points");

// The candidates' order (distance, caller index) as one 64-bit key: distances
// are non-negative, so their bits order as their values do.
__device__ __forceinline__ uint64_t knn_key(float d2, int32_t j) {
    return ((uint64_t)__float_as_uint(d2) << 32) | (uint32_t)j;
}

// the record of caller index i, at place w of the index
__device__ __forceinline__ void store_record(const ScanRecords& R, int i, int w, const float4 r0, const float4 r1,
                                             const float4 r2) {
    const auto put = [&](float4* __restrict__ to, int at) {
        to[3 * at] = r0;
        to[3 * at + 1] = r1;
        to[3 * at + 2] = r2;
    };
    put(R.caller, i);
    put(R.index, w);
    if (R.walk) put(R.walk, R.wpos[i]);
}

// The loops that are not unrolled keep the code short: a launch over a few
// hundred points spends its time fetching instructions for the first time.
template <int H>   // list entries per lane
__global__ __launch_bounds__(kB) void k_scan_knn_cov(const float* __restrict__ xyz, ScanIndex X, int n, int k,
                                                     float eps, ScanRecords R, uint64_t* __restrict__ stamp_end) {
    constexpr int kPer = kB / kQLanes;
    __shared__ float nbr[kPer][H * kQLanes][3];
    __shared__ double cov[kPer][7];   // 6 and a pad
    const int grp = threadIdx.x / kQLanes, gl = threadIdx.x % kQLanes;
    const int w = blockIdx.x * kPer + grp;
    const bool active = w < n;   // uniform over the point's lanes
    const float4 p4 = X.pts[active ? w : 0];
    const float3 pi = make_float3(p4.x, p4.y, p4.z);
    const int kk = min(k, n - 1);
    uint64_t best[H];
#pragma unroll
    for (int m = 0; m < H; ++m) best[m] = knn_key(__builtin_inff(), 0x7FFFFFFF);
    // lists needed per lane for the seed below to bound the kk-th distance
    const int mb = kk > kQLanes ? 1 : 0;
    float bound = __builtin_inff();
    // Seed the bound from the (up to 64) points nearest to this one in walk
    // order: every lane measures up to four of them with the arithmetic of the
    // search: 16 (mb + 1) >= kk of them lie at or below the largest of the lanes'
    // best (second best for mb = 1), and so do the kk nearest.  Candidates (and
    // boxes) above the bound are never needed.  (Without a seed 8192 points take
    // 60 us: the first candidates all go through the list.)
    const int nseed = min(4, (n - 1) / kQLanes);
    if (nseed > mb) {
        const int start = max(0, min(w - kQLanes * nseed / 2, n - 1 - kQLanes * nseed));
        float s0 = __builtin_inff(), s1 = __builtin_inff();
        for (int r = 0; r < nseed; ++r) {
            int q = start + kQLanes * r + gl;
            q += q >= w ? 1 : 0;
            const float d2 = mp_point_d2(X.pts[min(q, n - 1)], pi);
            s1 = fminf(s1, fmaxf(s0, d2));
            s0 = fminf(s0, d2);
        }
        bound = mp_row_max(mb >= 1 ? s1 : s0);
    }
    // the boxes, nearest first and walked by the whole wave: a group without
    // work idles along
    const int batches = (X.supers + kQLanes - 1) / kQLanes;
    int batch = w / (kIdxThreads * kQLanes);   // its own first
    for (int t = 0; t < batches; ++t, batch = batch + 1 < batches ? batch + 1 : 0) {
        const int sup = batch * kQLanes + gl;
        uint32_t sk = mp_box_key(active && sup < X.supers, X.super + 2 * min(sup, X.supers - 1), pi, gl);
        for (;;) {
            const uint32_t su = mp_row_min_u32(sk);
            const bool go = su != ~0u && __uint_as_float(su & ~15u) <= bound;
            if (!__any(go)) break;
            if ((su & 15u) == (uint32_t)gl) sk = ~0u;
            const int blk0 = (batch * kQLanes + (int)(su & 15u)) * kScanFan;
            const int blk = blk0 + gl;
            uint32_t bk = mp_box_key(go && blk < X.blocks, X.box + 2 * min(blk, X.blocks - 1), pi, gl);
            for (;;) {
                const uint32_t bl = mp_row_min_u32(bk);
                const bool gob = bl != ~0u && __uint_as_float(bl & ~15u) <= bound;
                if (!__any(gob)) break;
                if ((bl & 15u) == (uint32_t)gl) bk = ~0u;
                const int q0 = gob ? (blk0 + (int)(bl & 15u)) * kScanBlock + gl : n;
                float4 next = X.pts[min(q0, n - 1)];
#pragma unroll 1
                for (int r = 0; r < kScanBlock / kQLanes; ++r) {
                    const int q = q0 + kQLanes * r;
                    const float4 c = next;
                    next = X.pts[min(q + kQLanes, n - 1)];
                    const float d2 = mp_point_d2(c, pi);
                    const uint64_t key = knn_key(d2, __float_as_int(c.w));
                    uint32_t hits = mp_row_ballot(q < n && q != w && d2 <= bound);
                    if (!__any(hits != 0)) continue;
                    do {
                        const uint64_t got = __shfl((unsigned long long)key, hits ? __builtin_ctz(hits) : 0, kQLanes);
                        const uint64_t in = hits ? got : ~0ull;
                        hits &= hits - 1;
                        const uint64_t before = mp_row_shr(best[0], 0);
                        if (H > 1) {   // the upper 16 first: their first lane follows the lower ones' last
                            const uint64_t last = __shfl((unsigned long long)best[0], kQLanes - 1, kQLanes);
                            const uint64_t b1 = mp_row_shr(best[H - 1], last);
                            best[H - 1] = in < b1 ? b1 : (in < best[H - 1] ? in : best[H - 1]);
                        }
                        best[0] = in < before ? before : (in < best[0] ? in : best[0]);
                    } while (__any(hits != 0));
                    float far = gl < kk ? __uint_as_float((uint32_t)(best[0] >> 32)) : 0.0f;
                    if (H > 1) far = fmaxf(far, kQLanes + gl < kk ? __uint_as_float((uint32_t)(best[H - 1] >> 32)) : 0.0f);
                    bound = fminf(bound, mp_row_max(far));
                }
            }
        }
    }
#pragma unroll
    for (int m = 0; m < H; ++m) {
        const int a = m * kQLanes + gl;
        if (active && a < kk) {
            const int j = (int32_t)(uint32_t)best[m];
            nbr[grp][a][0] = xyz[3 * j];
            nbr[grp][a][1] = xyz[3 * j + 1];
            nbr[grp][a][2] = xyz[3 * j + 2];
        }
    }
    __syncthreads();
    const bool given = kk + 1 >= 5;   // fewer points give the identity
    const double dn = (double)(kk + 1);
    if (given) {
        // sums in list order, the point itself first
        const auto axis = [](const float3& v, int a) { return a == 0 ? v.x : (a == 1 ? v.y : v.z); };
        const int x = min(gl, 2);
        double sm = (double)axis(pi, x);
#pragma unroll 2
        for (int a = 0; a < kk; ++a) sm = sm + (double)nbr[grp][a][x];
        sm = sm / dn;
        const double mu[3] = {__shfl(sm, 0, kQLanes), __shfl(sm, 1, kQLanes), __shfl(sm, 2, kQLanes)};
        const int r = gl < 3 ? 0 : (gl < 5 ? 1 : 2), c = gl < 3 ? gl : (gl < 5 ? gl - 2 : 2);
        const double mr = r == 0 ? mu[0] : (r == 1 ? mu[1] : mu[2]), mc = c == 0 ? mu[0] : (c == 1 ? mu[1] : mu[2]);
        double S = 0.0;
        double d0 = (double)axis(pi, r) - mr, d1 = (double)axis(pi, c) - mc;
        S += d0 * d1;
#pragma unroll 2
        for (int a = 0; a < kk; ++a) {
            d0 = (double)nbr[grp][a][r] - mr;
            d1 = (double)nbr[grp][a][c] - mc;
            S += d0 * d1;
        }
        if (gl < 6) cov[grp][gl] = S / dn;
    }
    __syncthreads();
    const int wl = blockIdx.x * kPer + threadIdx.x;
    if (threadIdx.x < kPer && wl < n) {
        double c6[6] = {1, 0, 0, 1, 0, 1};
        if (given) {
            const double* S = cov[threadIdx.x];
            double A[9] = {S[0], S[1], S[2], S[1], S[3], S[4], S[2], S[4], S[5]};
            double nv[3];
            jacobi_min_vec(A, nv);
            const double a = 1.0 - (double)eps;
            c6[0] = 1.0 - a * nv[0] * nv[0];
            c6[1] = -a * nv[0] * nv[1];
            c6[2] = -a * nv[0] * nv[2];
            c6[3] = 1.0 - a * nv[1] * nv[1];
            c6[4] = -a * nv[1] * nv[2];
            c6[5] = 1.0 - a * nv[2] * nv[2];
        }
        const float4 p = X.pts[wl];
        const int i = __float_as_int(p.w);
        const float4 r0 = make_float4(p.x, p.y, p.z, (float)c6[0]);
        const float4 r1 = make_float4((float)c6[1], (float)c6[2], (float)c6[3], (float)c6[4]);
        const float4 r2 = make_float4((float)c6[5], 0.0f, 0.0f, 0.0f);
        store_record(R, i, wl, r0, r1, r2);
    }
    stamp_last(stamp_end);
}

__global__ void k_scan_given_cov(const float* __restrict__ cov, ScanIndex X, int n, ScanRecords R,
                                 uint64_t* __restrict__ stamp_end) {
    const int w = blockIdx.x * blockDim.x + threadIdx.x;
    if (w < n) {
        const float4 p = X.pts[w];
        const int i = __float_as_int(p.w);
        const float* c = cov + 6 * (size_t)i;
        const float4 r0 = make_float4(p.x, p.y, p.z, c[0]), r1 = make_float4(c[1], c[2], c[3], c[4]);
        const float4 r2 = make_float4(c[5], 0.0f, 0.0f, 0.0f);
        store_record(R, i, w, r0, r1, r2);
    }
    stamp_last(stamp_end);
}

__device__ inline uint32_t spread10(uint32_t v) {
    v &= 0x3FFu;
    v = (v | (v << 16)) & 0x030000FFu;
    v = (v | (v << 8)) & 0x0300F00Fu;
    v = (v | (v << 4)) & 0x030C30C3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

// Check, walk keys and verdict of an uploaded scan.  What bounds it: launches
// and the host's wait.  The verdict goes straight to pinned host memory, so that
// the host can go on while the device sorts.
constexpr int kChk = 1024;

constexpr int kOwnOrderMin = 3072;   // points, see scan_unfit

struct ScanMin {
    float lo[6];   // minimum corner of the points, negated maximum corner
    bool bad;
};

// of the points [from, to), by a workgroup of kChk
__device__ __forceinline__ ScanMin scan_min(const ScanPrep& A, int from, int to) {
    __shared__ float red[7][kChk / 64];
    constexpr float kInf = __builtin_inff();
    ScanMin M{{kInf, kInf, kInf, kInf, kInf, kInf}, false};
    const int corners = A.n < kOwnOrderMin ? 3 : 6;   // (scan_unfit asks for the maximum)
    for (int i = from + threadIdx.x; i < to; i += kChk) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float v = A.xyz[3 * i + a];
            M.bad |= !__builtin_isfinite(v);
            M.lo[a] = fminf(M.lo[a], v);
            if (corners == 6) M.lo[3 + a] = fminf(M.lo[3 + a], -v);
        }
        if (A.cov)
#pragma unroll
            for (int a = 0; a < 6; ++a) M.bad |= !__builtin_isfinite(A.cov[6 * (size_t)i + a]);
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int a = 0; a < 6; ++a)
        if (a < corners) M.lo[a] = wave_min(M.lo[a]);
    const bool any = __any(M.bad);
    if (lane == 0) {
        for (int a = 0; a < 6; ++a) red[a][wave] = M.lo[a];
        red[6][wave] = any ? 1.0f : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int a = 0; a < 6; ++a)
        if (a < corners) M.lo[a] = wave_min(red[a][lane % (kChk / 64)]);
    M.bad = __any(red[6][lane % (kChk / 64)] != 0.0f);
    return M;
}

// 30-bit Morton (Z-order) key of the point's cell (1024 cells per axis from
// the box corner, clamped) and the identity permutation
__device__ __forceinline__ void scan_key(const ScanPrep& A, const float lo[3], int i) {
    uint32_t c[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float q = floorf((A.xyz[3 * i + a] - lo[a]) * A.inv_cell);
        c[a] = (uint32_t)fminf(fmaxf(q, 0.0f), 1023.0f);
    }
    A.key[i] = spread10(c[0]) | (spread10(c[1]) << 1) | (spread10(c[2]) << 2);
    A.idx[i] = i;
}

// Whether the cells of the walk order, which the index takes over, do not tell
// neighbours apart: the scan reaches beyond the 1024 cells of an axis (what lies
// there is clamped into the last one), or has more than a block of points to a
// cell even if it fills its box.  Small scans keep the walk order: their index has
// few boxes in any case (microseconds of an upload and of ten iterations of
// odometry, points in random order and one 8 km off, walk order / own order: 2000
// points 83 and 284 / 101 and 202; in the order of a turning sensor 69 and 187 /
// 102 and 204; 4000 points 117 and 409 / 123 and 236, and 100 and 261 / 128 and 226).
__device__ __forceinline__ bool scan_unfit(const ScanPrep& A, const float lo[6]) {
    if (A.n < kOwnOrderMin) return false;
    float cells = 1.0f, most = 0.0f;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float c = floorf((-lo[3 + a] - lo[a]) * A.inv_cell) + 1.0f;
        cells *= c;
        most = fmaxf(most, c);
    }
    return most > 1024.0f || cells * (float)kScanBlock < (float)A.n;
}

__device__ __forceinline__ void scan_verdict(const ScanPrep& A, const float lo[6], bool bad) {
    *A.start = (uint64_t)wall_clock64();
    const uint32_t word = 4 * A.seq + (scan_unfit(A, lo) ? 2u : 0u) + (bad ? 1u : 0u);
    __hip_atomic_store(A.verdict, word, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// scans of up to kPrepOne points, in one workgroup
__global__ __launch_bounds__(kChk) void k_scan_prep(ScanPrep A) {
    const ScanMin M = scan_min(A, 0, A.n);
    if (threadIdx.x == 0) scan_verdict(A, M.lo, M.bad);
    for (int i = threadIdx.x; i < A.n; i += kChk) scan_key(A, M.lo, i);
}

// larger ones: a workgroup per kChk points, whose results every workgroup of
// the keys reduces (up to 64 of them, one a lane)
__global__ __launch_bounds__(kChk) void k_scan_check(ScanPrep A) {
    const ScanMin M = scan_min(A, blockIdx.x * kChk, min(A.n, ((int)blockIdx.x + 1) * kChk));
    if (threadIdx.x == 0) {
        A.part[2 * blockIdx.x] = make_float4(M.lo[0], M.lo[1], M.lo[2], M.bad ? 1.0f : 0.0f);
        A.part[2 * blockIdx.x + 1] = make_float4(M.lo[3], M.lo[4], M.lo[5], 0.0f);
    }
}

__global__ __launch_bounds__(256) void k_scan_keys(ScanPrep A) {
    const int nb = (A.n + kChk - 1) / kChk;
    const int b = min((int)(threadIdx.x & 63), nb - 1);
    const float4 p = A.part[2 * b];
    float lo[6] = {wave_min(p.x), wave_min(p.y), wave_min(p.z)};
    const bool bad = __any(p.w != 0.0f);
    if (blockIdx.x == 0) {
        const float4 u = A.part[2 * b + 1];
        lo[3] = wave_min(u.x);
        lo[4] = wave_min(u.y);
        lo[5] = wave_min(u.z);
        if (threadIdx.x == 0) scan_verdict(A, lo, bad);
    }
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < A.n) scan_key(A, lo, i);
}

// ------------------------------------------------------------ an index's own order
// Morton keys on cells that grow with the distance from the scan's middle, for
// scans that do not fit the walk order's cells whatever its points' spread: per
// axis the middle is the median of 64 points taken evenly, the unit s the largest
// axis's median distance from it, and a cell log2(1 + 16 |d| / s) / 21 wide, 1024
// of them, up to 10^6 s away.  No result depends on the order but that of the
// odometry's sums over the current scan.
//
// What bounds it: a sort and a launch more in the upload.  Milliseconds of an
// upload and of ten iterations of odometry, 65,536 points in random order, all
// points against all, walk order, own order: one of them 8 km off 4.5 and 8.4,
// 3.1 and 26.8, 0.32 and 0.85; 1000 m wide 4.5 and 8.4, 2.6 and 9.7, 0.33 and
// 0.79; 5 m wide under 5 m cells 4.5 and 8.4, 2.6 and 23.8, 0.30 and 0.77.  8192
// points, one off, 0.39 and 0.42, 0.19 and 0.71, 0.16 and 0.26.
__device__ __forceinline__ float wave_median(float v) {   // of a wave's 64 values
    const int lane = threadIdx.x & 63;
    int below = 0;
    for (int j = 0; j < 64; ++j) {
        const float o = __shfl(v, j);
        below += o < v || (o == v && j < lane) ? 1 : 0;
    }
    const uint64_t at = __ballot(below == 32);   // one lane
    return __shfl(v, at ? __builtin_ctzll(at) : 0);
}

__global__ __launch_bounds__(256) void k_index_keys(ScanPrep A, uint32_t* __restrict__ key, int32_t* __restrict__ perm,
                                                    int32_t* __restrict__ wpos) {
    const int64_t j = (int64_t)(threadIdx.x & 63) * A.n / 64;
    float mid[3], s = 0.0f;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float v = A.xyz[3 * j + a];
        mid[a] = wave_median(v);
        s = fmaxf(s, wave_median(fabsf(v - mid[a])));
    }
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= A.n) return;
    uint32_t c[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float d = A.xyz[3 * i + a] - mid[a];
        const float q = 512.0f + copysignf(21.0f * __log2f(1.0f + 16.0f * fabsf(d) / s), d);
        c[a] = (uint32_t)fminf(fmaxf(q, 0.0f), 1023.0f);   // (s = 0: the axis in two halves; NaN: 0)
    }
    key[i] = spread10(c[0]) | (spread10(c[1]) << 1) | (spread10(c[2]) << 2);
    perm[i] = i;
    wpos[A.idx[i]] = i;   // (A.idx: the walk order, sorted)
}

}  // namespace

size_t mp_scan_index_bytes(int32_t n) {
    const size_t b = (size_t)((n + kScanBlock - 1) / kScanBlock), u = (size_t)((n + kIdxThreads - 1) / kIdxThreads);
    return sizeof(float4) * ((size_t)n + 2 * b + 2 * u);
}

ScanIndex mp_scan_index(const DevMem& mem, int32_t n) {
    ScanIndex X;
    X.n = n;
    X.blocks = (n + kScanBlock - 1) / kScanBlock;
    X.supers = (n + kIdxThreads - 1) / kIdxThreads;
    X.pts = mem.as<float4>();
    X.box = X.pts + n;
    X.super = X.box + 2 * (size_t)X.blocks;
    return X;
}

void mp_scan_records(const float* xyz, const float* cov6, const int32_t* perm, int32_t n, int32_t k, float eps,
                     const ScanIndex& X, const ScanRecords& R, const uint64_t* start, uint64_t* stamps, hipStream_t s) {
    if (n <= 0) return;
    if (k > kKMax) mp_throw(MP_E_UNSUPPORTED, "scan_k above %d", kKMax);
    k_scan_index<<<X.supers, kIdxThreads, 0, s>>>(xyz, perm, n, X, start, stamps);
    MP_CHECK_LAUNCH();
    if (cov6) {
        k_scan_given_cov<<<(n + 255) / 256, 256, 0, s>>>(cov6, X, n, R, stamps + 1);
    } else {
        constexpr int per = kB / kQLanes;
        const unsigned grid = (unsigned)((n + per - 1) / per);
        if (k <= kQLanes) k_scan_knn_cov<1><<<grid, kB, 0, s>>>(xyz, X, n, k, eps, R, stamps + 1);
        else k_scan_knn_cov<2><<<grid, kB, 0, s>>>(xyz, X, n, k, eps, R, stamps + 1);
    }
    MP_CHECK_LAUNCH();
}

void mp_scan_walk_order(ScanPrep A, float cell, uint32_t* keys_alt, int32_t* perm_alt, DevMem& scratch,
                        hipStream_t s) {
    A.inv_cell = 1.0f / cell;
    if (A.n <= kPrepOne) {
        k_scan_prep<<<1, kChk, 0, s>>>(A);
    } else {
        k_scan_check<<<(A.n + kChk - 1) / kChk, kChk, 0, s>>>(A);
        k_scan_keys<<<(A.n + 255) / 256, 256, 0, s>>>(A);
    }
    MP_CHECK_LAUNCH();
    if (mp_sort_is_small(A.n)) mp_sort_small(SmSortArgs{A.key, A.key, A.idx, nullptr, nullptr, nullptr, A.n, 30, nullptr}, s);
    else mp_radix_sort_u32(A.key, A.idx, keys_alt, perm_alt, A.n, 30, scratch, s);
}

void mp_scan_index_order(const ScanPrep& A, uint32_t* keys_alt, int32_t* perm, int32_t* perm_alt, int32_t* wpos,
                         DevMem& scratch, hipStream_t s) {
    k_index_keys<<<(A.n + 255) / 256, 256, 0, s>>>(A, A.key, perm, wpos);
    MP_CHECK_LAUNCH();
    if (mp_sort_is_small(A.n)) mp_sort_small(SmSortArgs{A.key, A.key, perm, nullptr, nullptr, nullptr, A.n, 30, nullptr}, s);
    else mp_radix_sort_u32(A.key, perm, keys_alt, perm_alt, A.n, 30, scratch, s);
}
