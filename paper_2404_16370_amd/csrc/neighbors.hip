// neighbors.hip -- LSH bucketing and the iterative neighbour-list refresh
// (Eq. 9-10 and Alg. 1, IterativeNeighborParticleSearch).
//
//   k_lsh        per particle: zeta = alpha W^K x_i + delta_i with the tangent
//                x_i = [log(R_L^T R_i); R_L^T (t_i - t_L)] (decoupled) or
//                log(T_LSH^-1 T_i) (coupled SE(3) logarithm),
//                cell = floor(zeta) (deterministic FP32), code =
//                hash6(cell) & (2^bits - 1).  T^LSH is drawn from Philox for
//                (frame, iteration) by one lane of a workgroup.  The SVGD update
//                leaves the codes of the iterations after the first.
//   sort         stable radix sort of (code, index)  -> buckets as runs
//   k_bucket_bounds  bucket head/end per sorted position (search of the runs);
//                sorts in one workgroup leave them themselves
//   k_refresh_row, k_refresh  16 lanes or one per particle (its sorted position
//                from a rank array): candidates = previous list U
//                window of up to C bucket-mates after the particle (cyclic in
//                its bucket); each ranked by q_ij = d^T W^K d (deterministic
//                FP32), the K-1 smallest (q, j) kept behind the particle itself
//                (row minima, or a register-resident insertion network);
//                k_ij = exp(-q_ij) cached for the SVGD update and the posterior
//                propagation.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "mp_det.hpp"
#include "mp_internal.hpp"
#include "mp_lsh.hpp"
#include "mp_many.hpp"
#include "mp_row.hpp"

namespace {

__global__ __launch_bounds__(256) void k_lsh(LshArgs A) {
    mp_write_stamp(A.stamp);
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (A.dyn) A.frame = A.dyn->frame;
    if (A.flags && i < 4) A.flags[i] = 0;
    __shared__ float sL[8];
    if (threadIdx.x == 0) lsh_draw(A, sL, blockIdx.x == 0);
    __syncthreads();
    if (i < A.n) lsh_code(A, sL, i, A.poses[2 * i], A.poses[2 * i + 1]);
}

// Position of every particle in the sorted order, and bucket head and end of
// every position: the run of equal codes around
// s, found by an exponential then binary search on each side (a bucket of m
// particles costs about 2 log2(m) reads per position).
__global__ void k_bucket_bounds(const uint32_t* __restrict__ sc, const int32_t* __restrict__ sorted, int n,
                                int32_t* __restrict__ head, int32_t* __restrict__ end, int32_t* __restrict__ rank,
                                uint64_t* __restrict__ stamp) {
    mp_write_stamp(stamp);
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    const int i = sorted[s];
    if (i >= 0 && i < n) rank[i] = s;
    const uint32_t c = sc[s];
    // left: lo is known to hold c, the first position holding c is in (lo - step, lo]
    int lo = s, step = 1;
    while (lo - step >= 0 && sc[lo - step] == c) {
        lo -= step;
        step <<= 1;
    }
    int a = max(lo - step, -1), b = lo;   // sc[a] != c (or a = -1), sc[b] == c
    while (b - a > 1) {
        const int mid = a + (b - a) / 2;
        if (sc[mid] == c) b = mid;
        else a = mid;
    }
    head[s] = b;
    // right: the last position holding c is in [hi, hi + step)
    int hi = s;
    step = 1;
    while (hi + step < n && sc[hi + step] == c) {
        hi += step;
        step <<= 1;
    }
    a = hi;
    b = min(hi + step, n);   // sc[a] == c, sc[b] != c (or b = n)
    while (b - a > 1) {
        const int mid = a + (b - a) / 2;
        if (sc[mid] == c) a = mid;
        else b = mid;
    }
    end[s] = b;
}

struct RefreshArgs {
    const float4* __restrict__ poses;
    const int32_t* __restrict__ sorted;
    const int32_t* __restrict__ rank;   // sorted position of each particle
    const int32_t* __restrict__ head;
    const int32_t* __restrict__ end;
    int32_t* __restrict__ nbr;    // K x N
    float* __restrict__ kval;     // K x N
    int32_t* __restrict__ cnt;    // N
    int32_t n, K, C;
    float sr, st;
    uint64_t* stamp;              // stage clock, or null
};

template <int KM>
struct TopK {
    float q[KM];
    int32_t j[KM];
    __device__ void init() {
#pragma unroll
        for (int m = 0; m < KM; ++m) {
            q[m] = __builtin_inff();
            j[m] = 0x7FFFFFFF;
        }
    }
    __device__ bool has(int32_t x) const {
        bool h = false;
#pragma unroll
        for (int m = 0; m < KM; ++m) h |= (j[m] == x);
        return h;
    }
    // keep the KM smallest (q, j) in ascending order
    __device__ void insert(float qv, int32_t jv) {
#pragma unroll
        for (int m = KM - 1; m >= 1; --m) {
            const bool lt_prev = (qv < q[m - 1]) || (qv == q[m - 1] && jv < j[m - 1]);
            const bool lt_cur = (qv < q[m]) || (qv == q[m] && jv < j[m]);
            const float nq = lt_prev ? q[m - 1] : (lt_cur ? qv : q[m]);
            const int32_t nj = lt_prev ? j[m - 1] : (lt_cur ? jv : j[m]);
            q[m] = nq;
            j[m] = nj;
        }
        const bool lt0 = (qv < q[0]) || (qv == q[0] && jv < j[0]);
        if (lt0) {
            q[0] = qv;
            j[0] = jv;
        }
    }
};

// rank[sorted[s]] = s, when no sort left it (an order set from outside)
__global__ void k_rank(const int32_t* __restrict__ sorted, int n, int32_t* __restrict__ rank) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    const int i = sorted[s];
    if (i >= 0 && i < n) rank[i] = s;
}

// One lane per particle, in particle order, so that the particle's pose, its
// old list and its new list and kernel values are read and written coalesced;
// its sorted position (rank) locates its bucket window.
template <int KM>
__global__ __launch_bounds__(256) void k_refresh(RefreshArgs A) {
    mp_write_stamp(A.stamp);
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= A.n) return;
    const int s = A.rank[i];
    if (s < 0 || s >= A.n || A.sorted[s] != i) return;
    const float4 qi4 = A.poses[2 * i], ti4 = A.poses[2 * i + 1];
    const mpdet::quat qi{qi4.x, qi4.y, qi4.z, qi4.w};
    const float3 ti = make_float3(ti4.x, ti4.y, ti4.z);
    TopK<KM> tk;
    tk.init();
    auto consider = [&](int32_t j) {
        if (j < 0 || j >= A.n || j == i || tk.has(j)) return;
        const float4 qj4 = A.poses[2 * j], tj4 = A.poses[2 * j + 1];
        const float qv = mpdet::qdist(qi, ti, mpdet::quat{qj4.x, qj4.y, qj4.z, qj4.w},
                                      make_float3(tj4.x, tj4.y, tj4.z), A.sr, A.st);
        tk.insert(qv, j);
    };
    // bucket window (Alg. 1 gather loop, capped at C mates)
    int h = A.head[s], e = A.end[s];
    if (!(h >= 0 && h <= s && s < e && e <= A.n)) {
        h = s;
        e = s + 1;
    }
    const int m = e - h;
    const int w = min(m - 1, A.C);
    for (int d = 1; d <= w; ++d) {
        int pos = s + d;
        if (pos >= e) pos -= m;
        consider(A.sorted[pos]);
    }
    // previous list (persists across iterations)
    for (int a = 1; a < A.K; ++a) consider(A.nbr[(size_t)a * A.n + i]);
    // write: the particle itself first, then the K-1 nearest others
    A.nbr[i] = i;
    A.kval[i] = 1.0f;
    int c = 1;
#pragma unroll
    for (int a = 0; a < KM; ++a) {
        if (a + 1 < A.K) {
            const bool ok = tk.j[a] != 0x7FFFFFFF;
            A.nbr[(size_t)(a + 1) * A.n + i] = ok ? tk.j[a] : -1;
            A.kval[(size_t)(a + 1) * A.n + i] = ok ? expf(-tk.q[a]) : 0.0f;
            c += ok ? 1 : 0;
        }
    }
    A.cnt[i] = c;
}

// The same refresh with 16 lanes per particle: lane l ranks candidates l, l +
// 16, ... (at most R of them: the window, then the old list), all their loads
// in flight together, and the K - 1 smallest (q, j) are then taken one by one
// as the minimum over the lanes.  A candidate found twice has one key and is
// taken once; a round of candidates that no lane of the wave has costs nothing
// (the nearly empty lists of spread particles: 98,304 35 -> 21 us, converged ones
// 50 -> 39).  With one lane per particle the candidates' loads follow one
// another, some 1 us each while few waves run.
constexpr int kRfLanes = 16;
constexpr int kRfMax = 98304;   // most particles

template <int R>
__device__ __forceinline__ void refresh_row(const RefreshArgs& A, int block) {
    const int gl = threadIdx.x % kRfLanes;
    const int i0 = block * (256 / kRfLanes) + threadIdx.x / kRfLanes;
    const int i = min(i0, A.n - 1);
    const int s = A.rank[i];
    const bool active = i0 < A.n && s >= 0 && s < A.n && A.sorted[max(0, min(s, A.n - 1))] == i;   // uniform over the row
    const float4 qi4 = A.poses[2 * i], ti4 = A.poses[2 * i + 1];
    const mpdet::quat qi{qi4.x, qi4.y, qi4.z, qi4.w};
    const float3 ti = make_float3(ti4.x, ti4.y, ti4.z);
    int h = active ? A.head[s] : 0, e = active ? A.end[s] : 1;
    if (!(h >= 0 && h <= s && s < e && e <= A.n)) {
        h = s;
        e = s + 1;
    }
    const int m = e - h;
    const int w = active ? min(m - 1, A.C) : 0;
    const int cands = active ? w + A.K - 1 : 0;
    const uint64_t none = ((uint64_t)0x7F800000u << 32) | 0x7FFFFFFFu;   // (infinity, no particle)
    int32_t jc[R];
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const int c = u * kRfLanes + gl;
        jc[u] = -1;
        if (c < w) {
            int pos = s + 1 + c;
            if (pos >= e) pos -= m;
            jc[u] = A.sorted[pos];
        } else if (c < cands) {
            jc[u] = A.nbr[(size_t)(c - w + 1) * A.n + i];
        }
    }
    uint64_t key[R];
    float4 qj[R], tj[R];
    bool ok[R], any[R];   // (any: uniform over the wave)
#pragma unroll
    for (int u = 0; u < R; ++u) {
        ok[u] = jc[u] >= 0 && jc[u] < A.n && jc[u] != i;
        any[u] = __any(ok[u]);
    }
#pragma unroll
    for (int u = 0; u < R; ++u) {
        if (!any[u]) continue;
        const int j = ok[u] ? jc[u] : i;
        qj[u] = A.poses[2 * j];
        tj[u] = A.poses[2 * j + 1];
    }
#pragma unroll
    for (int u = 0; u < R; ++u) {
        key[u] = none;
        if (!any[u]) continue;
        // q >= 0: its bits order as its values do (weights of -0 give a q of -0: + 0)
        const float qv = mpdet::qdist(qi, ti, mpdet::quat{qj[u].x, qj[u].y, qj[u].z, qj[u].w},
                                      make_float3(tj[u].x, tj[u].y, tj[u].z), A.sr, A.st);
        key[u] = ok[u] ? ((uint64_t)__float_as_uint(qv + 0.0f) << 32) | (uint32_t)jc[u] : none;
    }
    // entry r (behind the particle itself) ends up in lane r % 16
    uint64_t mine[2] = {none, none};
    int cnt = 1;
#pragma unroll 1
    for (int r = 0; r + 1 < A.K; ++r) {
        uint64_t v = key[0];
#pragma unroll
        for (int u = 1; u < R; ++u) v = key[u] < v ? key[u] : v;
        v = mp_row_min_u64(v);
        if (!__any(v < none)) break;   // no list of the wave goes on
        cnt += v < none ? 1 : 0;
        if (gl == (r & (kRfLanes - 1))) {
            if (r < kRfLanes) mine[0] = v;
            else mine[1] = v;
        }
#pragma unroll
        for (int u = 0; u < R; ++u) key[u] = key[u] == v ? none : key[u];
    }
    if (!active) return;
    if (gl == 0) {
        A.nbr[i] = i;
        A.kval[i] = 1.0f;
        A.cnt[i] = cnt;
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int r = b * kRfLanes + gl;
        if (r + 1 >= A.K) break;
        const bool ok = mine[b] < none;
        A.nbr[(size_t)(r + 1) * A.n + i] = ok ? (int32_t)(uint32_t)mine[b] : -1;
        A.kval[(size_t)(r + 1) * A.n + i] = ok ? expf(-__uint_as_float((uint32_t)(mine[b] >> 32))) : 0.0f;
    }
}

__global__ void k_reset_lists(int32_t* __restrict__ nbr, float* __restrict__ kval, int32_t* __restrict__ cnt,
                              float* __restrict__ prior, int32_t* __restrict__ sorted, int32_t* __restrict__ head,
                              int32_t* __restrict__ end, int n, int K) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    // identity order, one particle per bucket, until the first LSH pass
    sorted[i] = i;
    head[i] = i;
    end[i] = i + 1;
    nbr[i] = i;
    kval[i] = 1.0f;
    for (int a = 1; a < K; ++a) {
        nbr[(size_t)a * n + i] = -1;
        kval[(size_t)a * n + i] = 0.0f;
    }
    cnt[i] = 1;
    prior[i] = 1.0f / (float)n;
}

template <int R>
__global__ __launch_bounds__(256) void k_refresh_row(RefreshArgs A) {
    mp_write_stamp(A.stamp);
    refresh_row<R>(A, blockIdx.x);
}

template <int R>
__global__ __launch_bounds__(256) void k_refresh_row_many(Many<RefreshArgs> M) {
    int block;
    const RefreshArgs A = many_args(M, block);
    refresh_row<R>(A, block);
}

inline unsigned nblk(int64_t n, int b = 256) { return (unsigned)((n + b - 1) / b); }

}  // namespace

LshArgs mp_lsh_args(mp_filter f, uint32_t frame, uint32_t it) {
    LshArgs A;
    A.poses = f->poses[f->cur].as<float4>();
    A.codes = f->codes.as<uint32_t>();
    // the sort ping-pongs between (tmp_keys, tmp_vals) and (scodes, sorted);
    // start it on the side that makes its last pass land in (scodes, sorted)
    const bool odd = mp_radix_passes(f->n, f->p.lsh_bits) % 2 == 1;
    A.keys = odd ? f->tmp_keys.as<uint32_t>() : f->scodes.as<uint32_t>();
    A.idx = odd ? f->tmp_vals.as<int32_t>() : f->sorted.as<int32_t>();
    A.tlsh = f->tlsh.as<float>();
    A.n = f->n;
    A.mask = f->p.lsh_bits >= 32 ? 0xFFFFFFFFu : ((1u << f->p.lsh_bits) - 1u);
    A.frame = frame;
    A.it = it;
    A.ar = f->p.lsh_alpha * f->p.sigma_r;
    A.at = f->p.lsh_alpha * f->p.sigma_t;
    A.sl = f->p.lsh_sigma;
    A.coupled = f->p.lsh_tangent == MP_LSH_TANGENT_SE3 ? 1 : 0;
    for (int a = 0; a < 3; ++a) {
        A.lo[a] = f->lsh_lo[a];
        A.hi[a] = f->lsh_hi[a];
    }
    A.seed = f->p.seed;
    A.dyn = f->dyn;
    A.flags = nullptr;
    A.stamp = nullptr;
    return A;
}

void mp_launch_lsh(mp_filter f, uint32_t frame, uint32_t it, hipStream_t s) {
    LshArgs A = mp_lsh_args(f, frame, it);
    A.flags = mp_take_flags(f);
    A.stamp = mp_take_stamp(f);
    k_lsh<<<nblk(f->n), 256, 0, s>>>(A);
    MP_CHECK_LAUNCH();
}

static SmSortArgs small_sort_args(mp_filter f) {
    // the LSH kernel's buffers, see there
    const bool odd = mp_radix_passes(f->n, f->p.lsh_bits) % 2 == 1;
    return SmSortArgs{odd ? f->tmp_keys.as<uint32_t>() : f->scodes.as<uint32_t>(), f->scodes.as<uint32_t>(),
                      f->sorted.as<int32_t>(), f->head.as<int32_t>(), f->end.as<int32_t>(), f->rank.as<int32_t>(),
                      f->n, f->n > 1 ? f->p.lsh_bits : 0, nullptr};
}

void mp_launch_sort(mp_filter f, hipStream_t s) {
    const int n = f->n;
    f->rank_set = true;
    if (mp_sort_is_small(n)) {
        SmSortArgs A = small_sort_args(f);
        A.stamp = mp_take_stamp(f);
        mp_sort_small(A, s);
        return;
    }
    // stable sort of (code, index) from the buffers the LSH kernel filled;
    // the result lands in (scodes, sorted) with no copy
    const bool odd = mp_radix_passes(n, f->p.lsh_bits) % 2 == 1;
    uint64_t* stamp = mp_radix_passes(n, f->p.lsh_bits) > 0 ? mp_take_stamp(f) : nullptr;
    if (odd)
        mp_radix_sort_u32_inplace_parity(f->tmp_keys.as<uint32_t>(), f->tmp_vals.as<int32_t>(),
                                         f->scodes.as<uint32_t>(), f->sorted.as<int32_t>(), n, f->p.lsh_bits, f->hist,
                                         s, stamp);
    else
        mp_radix_sort_u32_inplace_parity(f->scodes.as<uint32_t>(), f->sorted.as<int32_t>(), f->tmp_keys.as<uint32_t>(),
                                         f->tmp_vals.as<int32_t>(), n, f->p.lsh_bits, f->hist, s, stamp);
    k_bucket_bounds<<<nblk(n), 256, 0, s>>>(f->scodes.as<uint32_t>(), f->sorted.as<int32_t>(), n,
                                            f->head.as<int32_t>(), f->end.as<int32_t>(), f->rank.as<int32_t>(),
                                            mp_take_stamp(f));
    MP_CHECK_LAUNCH();
}

static RefreshArgs refresh_args(mp_filter f, int window) {
    RefreshArgs A;
    A.stamp = nullptr;
    A.poses = f->poses[f->cur].as<float4>();
    A.sorted = f->sorted.as<int32_t>();
    A.rank = f->rank.as<int32_t>();
    A.head = f->head.as<int32_t>();
    A.end = f->end.as<int32_t>();
    A.nbr = f->nbr.as<int32_t>();
    A.kval = f->kval.as<float>();
    A.cnt = f->cnt.as<int32_t>();
    A.n = f->n;
    A.K = f->K;
    A.C = window < 0 ? f->p.window_c : window;
    A.sr = f->p.sigma_r;
    A.st = f->p.sigma_t;
    return A;
}

// candidates per lane of the row kernel, or 0: one lane per particle
static int refresh_rows(mp_filter f, int C) {
    // 16 lanes per particle while one lane each would leave most of the chip
    // waiting for its loads, and for windows whose candidates fit five a lane.
    // One lane / 16 lanes, K = 16 and window 32: 4096 particles 44 / 7.4 us, 65,536
    // 53 / 29, 98,304 60 / 39, 131,072 63 / 51, 262,144 83 / 96; spread over a hall,
    // whose lists are nearly empty, 32,768 20 / 9.3 us, 65,536 25 / 16, 98,304 29 / 21,
    // 262,144 52 / 58.  K = 8 and window 16 lose from 131,072 on: 23 / 25 spread.
    const int64_t cands = (int64_t)C + f->K - 1;
    if (f->n > kRfMax || cands > 5 * kRfLanes) return 0;
    return cands <= 2 * kRfLanes ? 2 : (cands <= 3 * kRfLanes ? 3 : 5);
}

void mp_launch_refresh(mp_filter f, hipStream_t s, int window) {
    if (!f->rank_set) {
        k_rank<<<nblk(f->n), 256, 0, s>>>(f->sorted.as<int32_t>(), f->n, f->rank.as<int32_t>());
        MP_CHECK_LAUNCH();
        f->rank_set = true;
    }
    RefreshArgs A = refresh_args(f, window);
    A.stamp = mp_take_stamp(f);
    const int R = refresh_rows(f, A.C);
    if (R) {
        const unsigned grid = nblk(f->n, 256 / kRfLanes);
        if (R == 2) k_refresh_row<2><<<grid, 256, 0, s>>>(A);
        else if (R == 3) k_refresh_row<3><<<grid, 256, 0, s>>>(A);
        else k_refresh_row<5><<<grid, 256, 0, s>>>(A);
    } else if (f->K <= 8) k_refresh<8><<<nblk(f->n), 256, 0, s>>>(A);
    else if (f->K <= 16) k_refresh<16><<<nblk(f->n), 256, 0, s>>>(A);
    else k_refresh<32><<<nblk(f->n), 256, 0, s>>>(A);
    MP_CHECK_LAUNCH();
}

void mp_many_sort(const std::vector<mp_filter>& fs, ManyTab& T, hipStream_t s) {
    std::vector<SmSortArgs> a;
    for (mp_filter f : fs) {
        f->rank_set = true;
        a.push_back(small_sort_args(f));
    }
    if (!a.empty()) mp_sort_small_many(a, T, s);
}

void mp_many_refresh(const std::vector<mp_filter>& fs, ManyTab& T, hipStream_t s) {
    for (int R : {2, 3, 5}) {
        std::vector<RefreshArgs> a;
        std::vector<int32_t> blocks;
        for (mp_filter f : fs)
            if (refresh_rows(f, f->p.window_c) == R) {
                a.push_back(refresh_args(f, -1));
                blocks.push_back((int32_t)nblk(f->n, 256 / kRfLanes));
            }
        if (a.empty()) continue;
        unsigned grid;
        const Many<RefreshArgs> M = many_table(T, a, blocks, grid);
        if (R == 2) k_refresh_row_many<2><<<grid, 256, 0, s>>>(M);
        else if (R == 3) k_refresh_row_many<3><<<grid, 256, 0, s>>>(M);
        else k_refresh_row_many<5><<<grid, 256, 0, s>>>(M);
        MP_CHECK_LAUNCH();
    }
}

bool mp_refresh_is_rows(mp_filter f) { return refresh_rows(f, f->p.window_c) != 0; }

void mp_launch_reset_lists(mp_filter f, hipStream_t s) {
    k_reset_lists<<<nblk(f->n), 256, 0, s>>>(f->nbr.as<int32_t>(), f->kval.as<float>(), f->cnt.as<int32_t>(),
                                               f->prior.as<float>(), f->sorted.as<int32_t>(), f->head.as<int32_t>(),
                                               f->end.as<int32_t>(), f->n, f->K);
    MP_CHECK_LAUNCH();
}
