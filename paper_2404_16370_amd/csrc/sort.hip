// sort.hip -- device-wide exclusive scan and stable radix sorts.
//
// The radix sorts distribute particles into LSH buckets (Alg. 1, distribute
// loop), order the scan points for the likelihood's walk and group map points
// by voxel.  Every pass handles one digit (8 to 10 bits; 4 in the sort of few keys)
// and is stable, so the sort is stable: equal keys keep ascending value order when the values start as
// 0..n-1.
//
// 32-bit keys (the per-iteration sorts) take a one-sweep form: one launch
// counts the digits of every pass at once, then each pass is one launch in
// which a workgroup ranks its 4096-key tile locally, publishes its digit
// counts, reads the counts of the tiles before it (a decoupled look-back:
// each tile publishes first its own count, then its inclusive prefix, and a
// tile adds its predecessors' counts until it reaches an inclusive prefix)
// and writes its keys to their sorted places through LDS.  Tiles take their
// index from a counter in the order they start, so every tile a workgroup
// waits for belongs to a workgroup that is already running and publishes
// without waiting on later tiles; the wait is bounded all the same.
//
// 64-bit keys (the one-time voxel grouping of a map build) take three
// launches per pass: per-tile digit histograms (LDS atomics), an exclusive
// scan of the digit-major histogram matrix, and a stable scatter in which the
// rank among lanes with the same digit comes from eight 64-lane ballots.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "mp_internal.hpp"
#include "mp_many.hpp"

namespace {

constexpr int kThreads = 256;
constexpr int kItems = 4;
constexpr int kTile = kThreads * kItems;

__device__ inline uint32_t wave_incl_scan(uint32_t v, int lane) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        uint32_t u = __shfl_up(v, d, 64);
        if (lane >= d) v += u;
    }
    return v;
}

// block-wide exclusive scan of one value per thread; returns the block total
__device__ inline uint32_t block_excl_scan(uint32_t v, uint32_t& excl) {
    __shared__ uint32_t wsum[kThreads / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t inc = wave_incl_scan(v, lane);
    if (lane == 63) wsum[w] = inc;
    __syncthreads();
    uint32_t base = 0, total = 0;
#pragma unroll
    for (int k = 0; k < kThreads / 64; ++k) {
        if (k < w) base += wsum[k];
        total += wsum[k];
    }
    excl = base + inc - v;
    __syncthreads();
    return total;
}

__global__ __launch_bounds__(kThreads) void k_scan_reduce(const uint32_t* __restrict__ in, int64_t n,
                                                          uint32_t* __restrict__ sums) {
    const int64_t base = (int64_t)blockIdx.x * kTile;
    uint32_t s = 0;
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const int64_t i = base + r * kThreads + threadIdx.x;
        if (i < n) s += in[i];
    }
    uint32_t ex;
    const uint32_t tot = block_excl_scan(s, ex);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// exclusive scan of each tile plus the tile's offset; in == out allowed
__global__ __launch_bounds__(kThreads) void k_scan_apply(const uint32_t* in, uint32_t* out, int64_t n,
                                                         const uint32_t* __restrict__ offsets,
                                                         uint32_t* __restrict__ total) {
    const int64_t base = (int64_t)blockIdx.x * kTile + (int64_t)threadIdx.x * kItems;
    uint32_t v[kItems];
    uint32_t s = 0;
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        const int64_t i = base + j;
        v[j] = i < n ? in[i] : 0u;
        s += v[j];
    }
    uint32_t ex;
    const uint32_t tot = block_excl_scan(s, ex);
    const uint32_t off = offsets ? offsets[blockIdx.x] : 0u;
    uint32_t run = off + ex;
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        const int64_t i = base + j;
        if (i < n) out[i] = run;
        run += v[j];
    }
    if (total && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *total = off + tot;
}

size_t scan_scratch_words(int64_t n) {
    size_t w = 0;
    while (n > kTile) {
        n = (n + kTile - 1) / kTile;
        w += (size_t)n;
    }
    return w;
}

void scan_rec(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* total, uint32_t* scratch, hipStream_t s) {
    if (n <= 0) {
        if (total) mp_fill_u32(total, 0u, 1, s);
        return;
    }
    if (n <= kTile) {
        k_scan_apply<<<1, kThreads, 0, s>>>(in, out, n, nullptr, total);
        MP_CHECK_LAUNCH();
        return;
    }
    const int64_t nb = (n + kTile - 1) / kTile;
    uint32_t* sums = scratch;
    k_scan_reduce<<<(unsigned)nb, kThreads, 0, s>>>(in, n, sums);
    MP_CHECK_LAUNCH();
    scan_rec(sums, sums, nb, nullptr, scratch + nb, s);
    k_scan_apply<<<(unsigned)nb, kThreads, 0, s>>>(in, out, n, sums, total);
    MP_CHECK_LAUNCH();
}

template <class K>
__global__ __launch_bounds__(kThreads) void k_radix_hist(const K* __restrict__ keys, int64_t n, int shift,
                                                         uint32_t* __restrict__ counts, int64_t nblocks) {
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kTile;
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const int64_t i = base + r * kThreads + threadIdx.x;
        if (i < n) atomicAdd(&h[(uint32_t)(keys[i] >> shift) & 255u], 1u);
    }
    __syncthreads();
    counts[(int64_t)threadIdx.x * nblocks + blockIdx.x] = h[threadIdx.x];
}

template <class K>
__global__ __launch_bounds__(kThreads) void k_radix_scatter(const K* __restrict__ kin, const int32_t* __restrict__ vin,
                                                            K* __restrict__ kout, int32_t* __restrict__ vout,
                                                            int64_t n, int shift, const uint32_t* __restrict__ offs,
                                                            int64_t nblocks) {
    __shared__ uint32_t run[256];
    __shared__ uint32_t wcnt[kThreads / 64][256];
    __shared__ uint32_t wpre[kThreads / 64][256];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    run[t] = offs[(int64_t)t * nblocks + blockIdx.x];
    const int64_t base = (int64_t)blockIdx.x * kTile;
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    for (int r = 0; r < kItems; ++r) {
#pragma unroll
        for (int j = 0; j < kThreads / 64; ++j) wcnt[j][t] = 0;
        __syncthreads();
        const int64_t i = base + r * kThreads + t;
        const bool valid = i < n;
        const K key = valid ? kin[i] : (K)0;
        const int32_t val = valid ? vin[i] : 0;
        const uint32_t d = (uint32_t)(key >> shift) & 255u;
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bb = __ballot(bit);
            peers &= bit ? bb : ~bb;
        }
        const uint64_t lower = peers & below;
        const uint32_t rank = (uint32_t)__popcll(lower);
        if (valid && lower == 0ull) wcnt[w][d] = (uint32_t)__popcll(peers);
        __syncthreads();
        uint32_t s = run[t];
#pragma unroll
        for (int j = 0; j < kThreads / 64; ++j) {
            wpre[j][t] = s;
            s += wcnt[j][t];
        }
        run[t] = s;
        __syncthreads();
        if (valid) {
            const uint32_t pos = wpre[w][d] + rank;
            kout[pos] = key;
            vout[pos] = val;
        }
        __syncthreads();
    }
}

// Sorts (keys, vals) in 8-bit passes, ping-ponging with the alt arrays.  With
// copy_back the result is always left in (keys, vals); without it the result
// stays where the last pass wrote it, (keys_alt, vals_alt) after an odd
// number of passes.
template <class K>
void radix_sort(K* keys, int32_t* vals, K* keys_alt, int32_t* vals_alt, int64_t n, int bits, DevMem& scratch,
                hipStream_t s, bool copy_back = true) {
    if (n <= 1 || bits <= 0) return;
    const int passes = (bits + 7) / 8;
    const int64_t nb = (n + kTile - 1) / kTile;
    const int64_t m = 256 * nb;
    scratch.ensure(sizeof(uint32_t) * (size_t)(2 * m + scan_scratch_words(m) + 16));
    uint32_t* counts = scratch.as<uint32_t>();
    uint32_t* offs = counts + m;
    uint32_t* sscr = offs + m;
    K* ka = keys;
    int32_t* va = vals;
    K* kb = keys_alt;
    int32_t* vb = vals_alt;
    for (int p = 0; p < passes; ++p) {
        const int shift = 8 * p;
        k_radix_hist<K><<<(unsigned)nb, kThreads, 0, s>>>(ka, n, shift, counts, nb);
        MP_CHECK_LAUNCH();
        scan_rec(counts, offs, m, nullptr, sscr, s);
        k_radix_scatter<K><<<(unsigned)nb, kThreads, 0, s>>>(ka, va, kb, vb, n, shift, offs, nb);
        MP_CHECK_LAUNCH();
        std::swap(ka, kb);
        std::swap(va, vb);
    }
    if (copy_back && ka != keys) {
        MP_HIP(hipMemcpyAsync(keys, ka, sizeof(K) * (size_t)n, hipMemcpyDeviceToDevice, s));
        MP_HIP(hipMemcpyAsync(vals, va, sizeof(int32_t) * (size_t)n, hipMemcpyDeviceToDevice, s));
    }
}

// ------------------------------------------------------------ one-sweep sort of 32-bit keys
constexpr int kOsThreads = 512;
constexpr int kOsWaves = kOsThreads / 64;
constexpr int kOsItems = 8;                      // keys per thread: a wave ranks 8 rounds of 64
constexpr int kOsTile = kOsThreads * kOsItems;   // 4096 keys per tile
constexpr int kOsWaveKeys = kOsTile / kOsWaves;  // 512 consecutive keys per wave
constexpr int kOsMaxPasses = 4;
constexpr int kOsMaxCounts = 2 * 1024;           // passes times digits, at most (see os_plan)
constexpr int kOsHistThreads = 1024;
constexpr int kOsHistKeys = 16;                  // consecutive keys per histogram thread and round
constexpr int kOsMaxHistBlocks = 64;
constexpr int kOsWindow = 16;                    // predecessor tiles read per look-back step
constexpr uint32_t kOsSpinLimit = 1u << 20;      // look-back steps without progress before giving up
// a tile's published word for one digit: flag in the top two bits, count below
constexpr uint32_t kStAgg = 1u << 30;            // the tile's own count
constexpr uint32_t kStInc = 2u << 30;            // the count of all keys up to and including the tile
constexpr uint32_t kStVal = (1u << 30) - 1u;
// scratch words: [0, 4) tile counters of the passes, [4] wait flag, then the
// published words [pass][tile][digit], then the histogram blocks' counts
// [block][pass][digit] in kOsMaxCounts words each
constexpr int kOsHead = 16;

__device__ inline uint32_t os_load(const uint32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void os_store(uint32_t* p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct OsHistArgs {
    const uint32_t* __restrict__ keys;
    int64_t n;
    int32_t passes, bits;            // bits per pass
    int32_t vec;                     // keys 16-byte aligned: read four at a time
    uint32_t* __restrict__ part;     // [gridDim.x][kOsMaxCounts]
    uint32_t* __restrict__ clear;    // counters, flag and published words: zeroed
    int64_t clear_words;
    uint64_t* stamp;                 // stage clock, or null
};

// Digit counts of every pass over all keys.  A thread takes 16 consecutive
// keys and adds runs of equal digits with one LDS atomic per run (keys of a
// converged filter share codes over long runs).
__global__ __launch_bounds__(kOsHistThreads) void k_os_hist(OsHistArgs A) {
    __shared__ uint32_t h[kOsMaxCounts];
    mp_write_stamp(A.stamp);
    const int counts = A.passes << A.bits;
    const uint32_t mask = (1u << A.bits) - 1u;
    const int64_t gt = (int64_t)blockIdx.x * kOsHistThreads + threadIdx.x;
    const int64_t gstride = (int64_t)gridDim.x * kOsHistThreads;
    for (int j = threadIdx.x; j < counts; j += kOsHistThreads) h[j] = 0;
    for (int64_t j = gt; j < A.clear_words; j += gstride) A.clear[j] = 0;
    __syncthreads();
    for (int64_t i0 = gt * kOsHistKeys; i0 < A.n; i0 += gstride * kOsHistKeys) {
        uint32_t k[kOsHistKeys];
        if (A.vec && i0 + kOsHistKeys <= A.n) {
            const uint4* q = reinterpret_cast<const uint4*>(A.keys + i0);
#pragma unroll
            for (int c = 0; c < kOsHistKeys / 4; ++c) {
                const uint4 v = q[c];
                k[4 * c] = v.x;
                k[4 * c + 1] = v.y;
                k[4 * c + 2] = v.z;
                k[4 * c + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int c = 0; c < kOsHistKeys; ++c) k[c] = i0 + c < A.n ? A.keys[i0 + c] : 0u;
        }
        const int cnt = (int)min<int64_t>(kOsHistKeys, A.n - i0);
        for (int p = 0; p < A.passes; ++p) {
            uint32_t cur = (k[0] >> (A.bits * p)) & mask, run = 1;
#pragma unroll
            for (int c = 1; c < kOsHistKeys; ++c) {
                const uint32_t d = (k[c] >> (A.bits * p)) & mask;
                if (c < cnt && d == cur) {
                    ++run;
                } else if (c < cnt) {
                    atomicAdd(&h[(p << A.bits) + cur], run);
                    cur = d;
                    run = 1;
                }
            }
            atomicAdd(&h[(p << A.bits) + cur], run);
        }
    }
    __syncthreads();
    for (int j = threadIdx.x; j < counts; j += kOsHistThreads) A.part[(size_t)blockIdx.x * kOsMaxCounts + j] = h[j];
}

struct OsScatterArgs {
    const uint32_t* __restrict__ kin;
    const int32_t* __restrict__ vin;
    uint32_t* __restrict__ kout;
    int32_t* __restrict__ vout;
    int64_t n;
    int32_t shift, pass, nhist;
    const uint32_t* __restrict__ part;   // [nhist][kOsMaxCounts]
    uint32_t* status;                    // this pass: [tiles][digits], zero at launch
    uint32_t* ticket;                    // this pass's tile counter, zero at launch
    uint32_t* wait_flag;                 // 1: a look-back gave up; 2: a key fell outside the output
};

// One pass over BITS-bit digits: the grid has exactly one workgroup per tile.
template <int BITS>
__global__ __launch_bounds__(kOsThreads) void k_os_scatter(OsScatterArgs A) {
    constexpr int D = 1 << BITS;
    constexpr int kPer = D > kOsThreads ? D / kOsThreads : 1;   // consecutive digits of a thread
    constexpr int kOwners = D / kPer;                           // threads that hold digits
    constexpr int kParts = D >= kOsThreads ? 1 : kOsThreads / D;   // threads that sum a digit's histogram blocks
    __shared__ uint32_t wc[kOsWaves][D];     // per-wave digit counts, then the waves' exclusive offsets
    __shared__ uint32_t sk[kOsTile];
    __shared__ int32_t sv[kOsTile];
    __shared__ uint32_t tstart[D];           // first local position of each digit in the tile
    __shared__ uint32_t gbase[D];            // global position of a digit's keys minus tstart
    __shared__ uint32_t htot[kParts][D];     // digit totals summed by the parts of the workgroup
    __shared__ uint32_t wsc[kOsWaves], wsg[kOsWaves];
    __shared__ uint32_t s_tile;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    if (t == 0) s_tile = atomicAdd(A.ticket, 1u);
    for (int j = t; j < kOsWaves * D; j += kOsThreads) (&wc[0][0])[j] = 0;
    __syncthreads();
    const uint32_t tile = s_tile;
    const int64_t tbase = (int64_t)tile * kOsTile;
    const int64_t wbase = tbase + w * kOsWaveKeys;
    uint32_t key[kOsItems], lr[kOsItems];
    int32_t val[kOsItems];
#pragma unroll
    for (int r = 0; r < kOsItems; ++r) {
        const int64_t i = wbase + r * 64 + lane;
        key[r] = i < A.n ? A.kin[i] : 0u;
        val[r] = i < A.n ? A.vin[i] : 0;
    }
    // digit totals of this pass over all keys, from the histogram blocks: each
    // part of the workgroup sums its share of them (loads in flight together)
    {
        constexpr int kShare = kOsMaxHistBlocks / 2;
        const int part = kParts > 1 ? t / D : 0;
        for (int d = t % D; d < D; d += kOsThreads) {
            uint32_t sum = 0;
            for (int b0 = 0; b0 < A.nhist; b0 += kShare * kParts) {
                uint32_t pv[kShare];
#pragma unroll
                for (int b = 0; b < kShare; ++b) {
                    const int blk = b0 + kParts * b + part;
                    pv[b] = blk < A.nhist ? A.part[(size_t)blk * kOsMaxCounts + (A.pass << BITS) + d] : 0u;
                }
#pragma unroll
                for (int b = 0; b < kShare; ++b) sum += pv[b];
            }
            htot[part][d] = sum;
        }
    }
    // rank of each key among the keys of its wave with the same digit, in
    // key order: the lanes of a round sharing the digit (a ballot per bit), plus
    // the wave's running count of that digit from earlier rounds
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
    for (int r = 0; r < kOsItems; ++r) {
        const bool valid = wbase + r * 64 + lane < A.n;
        const uint32_t d = (key[r] >> A.shift) & (D - 1u);
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < BITS; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bb = __ballot(bit);
            peers &= bit ? bb : ~bb;
        }
        const uint32_t rk = (uint32_t)__popcll(peers & below);
        const uint32_t b0 = wc[w][d];
        if (valid && rk == 0) wc[w][d] = b0 + (uint32_t)__popcll(peers);
        lr[r] = b0 + rk;
    }
    __syncthreads();
    uint32_t cnt[kPer], tot[kPer], incc = 0, incg = 0;
    if (t < kOwners) {
        uint32_t sumc = 0, sumg = 0;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int d = t * kPer + j;
            tot[j] = 0;
            for (int part = 0; part < kParts; ++part) tot[j] += htot[part][d];
            cnt[j] = 0;
            for (int v = 0; v < kOsWaves; ++v) {
                const uint32_t c = wc[v][d];
                wc[v][d] = cnt[j];
                cnt[j] += c;
            }
            os_store(A.status + (size_t)tile * D + d, (tile == 0 ? kStInc : kStAgg) | cnt[j]);
            sumc += cnt[j];
            sumg += tot[j];
        }
        incc = wave_incl_scan(sumc, lane);
        incg = wave_incl_scan(sumg, lane);
        if (lane == 63) {
            wsc[w] = incc;
            wsg[w] = incg;
        }
        incc -= sumc;   // exclusive
        incg -= sumg;
    }
    __syncthreads();
    if (t < kOwners) {
        for (int v = 0; v < w; ++v) {
            incc += wsc[v];
            incg += wsg[v];
        }
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int d = t * kPer + j;
            const uint32_t ts = incc;   // tile-local start of digit d
            const uint32_t gs = incg;   // global start of digit d
            incc += cnt[j];
            incg += tot[j];
            // keys of digit d in the tiles before this one
            uint32_t excl = 0;
            int64_t tp = (int64_t)tile - 1;
            uint32_t idle = 0;
            while (tp >= 0) {
                uint32_t st[kOsWindow];
#pragma unroll
                for (int k = 0; k < kOsWindow; ++k)
                    st[k] = tp - k >= 0 ? os_load(A.status + (size_t)(tp - k) * D + d) : kStInc;
                int used = 0;
                bool done = false;
#pragma unroll
                for (int k = 0; k < kOsWindow; ++k) {
                    if (done || used < k) continue;              // stopped earlier in the window
                    const uint32_t sw = st[k];
                    if ((sw & ~kStVal) == 0u) continue;          // not published yet: read again from here
                    excl += sw & kStVal;
                    used = k + 1;
                    done = (sw & kStInc) != 0u;
                }
                if (done) break;
                tp -= used;
                if (used == 0) {
                    if (++idle > kOsSpinLimit) {
                        os_store(A.wait_flag, 1u);
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
            }
            if (tile > 0) os_store(A.status + (size_t)tile * D + d, kStInc | (excl + cnt[j]));
            tstart[d] = ts;
            gbase[d] = gs + excl - ts;
        }
    }
    __syncthreads();
    // keys to their sorted places in the tile
#pragma unroll
    for (int r = 0; r < kOsItems; ++r) {
        if (wbase + r * 64 + lane < A.n) {
            const uint32_t d = (key[r] >> A.shift) & (D - 1u);
            const uint32_t lp = tstart[d] + wc[w][d] + lr[r];
            sk[lp] = key[r];
            sv[lp] = val[r];
        }
    }
    __syncthreads();
    const int64_t tn = min<int64_t>(kOsTile, A.n - tbase);
#pragma unroll
    for (int r = 0; r < kOsItems; ++r) {
        const int j = r * kOsThreads + t;
        if (j < tn) {
            const uint32_t kk = sk[j];
            const uint32_t pos = gbase[(kk >> A.shift) & (D - 1u)] + (uint32_t)j;
            // a pass whose input is not a permutation of the counted keys (the
            // keys changed under the sort) could place a key past the end:
            // such keys are dropped and the sort flagged
            if ((int64_t)pos < A.n) {
                A.kout[pos] = kk;
                A.vout[pos] = sv[j];
            } else {
                os_store(A.wait_flag, 2u);
            }
        }
    }
}

// inclusive sum over the wave's lanes (all active): within rows of 16, then
// the rows' totals carried on
__device__ __forceinline__ uint32_t wave_scan_dpp(uint32_t v) {
    auto step = [&](auto ctrl, auto rows) {
        v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, decltype(rows)::value, 0xF, true);
    };
    step(std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xF>{});   // row_shr:1
    step(std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xF>{});
    step(std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xF>{});
    step(std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xF>{});
    step(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xA>{});   // row_bcast:15 into rows 1, 3
    step(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xC>{});   // row_bcast:31 into rows 2, 3
    return v;
}

// ------------------------------------------------------------ sort of few keys in one workgroup
// Up to kSmMax keys stay in the LDS of one workgroup through all passes, 4
// bits at a time: a thread counts the digits of its ITEMS consecutive keys in
// counters of its own, one scan over (digit, thread) turns the counts into
// places, and the thread hands the places out in key order.  For bucket sorts
// the same launch writes every position's bucket bounds and every value's
// position.
//
// What bounds it: LDS latency and the barriers of a pass, about 2 us each, and
// one CU's loads and stores.  With bounds and positions, 20-bit keys: 256 keys
// 7 us, 4096 15 us, 8000 23 us; the one-sweep sort and its bounds kernel, 27
// to 32 us and five launches whatever the count below 16,384 (where one
// workgroup took 64 us).
constexpr int kSmThreads = 1024;
constexpr int kSmItems = 8;                      // most keys per thread
constexpr int kSmMax = kSmThreads * kSmItems;
constexpr int kSmBits = 4;
constexpr int kSmDigits = 1 << kSmBits;          // one thread scans as many counters
static_assert(kSmDigits == 16, "a thread's share of the scan is two 16-byte words of 16-bit counters");
static_assert(4 * kSmItems <= 2 * kSmDigits, "heads and ends fit the counters");

template <int ITEMS, int T = kSmThreads>   // keys per thread, threads
__device__ __forceinline__ void sort_small(const SmSortArgs& A) {
    __shared__ __attribute__((aligned(16))) uint32_t sk[T * ITEMS];
    __shared__ __attribute__((aligned(16))) uint16_t sv[T * ITEMS];   // index of the key among the inputs
    __shared__ __attribute__((aligned(16))) uint32_t cnt[kSmDigits * T / 2];   // 16-bit counters [digit][thread]
    __shared__ uint32_t wsum[T / 64];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    for (int i = t; i < T * ITEMS; i += T) {
        sk[i] = i < A.n ? A.kin[i] : 0u;
        sv[i] = (uint16_t)i;
    }
    uint4* scan = reinterpret_cast<uint4*>(cnt) + 2 * t;   // this thread's share of the scan: 16 counters
    for (int shift = 0; shift < A.bits; shift += kSmBits) {
        scan[0] = make_uint4(0, 0, 0, 0);
        scan[1] = make_uint4(0, 0, 0, 0);
        __syncthreads();
        uint32_t key[ITEMS];
        uint16_t val[ITEMS];
        uint32_t pos[ITEMS];
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            key[r] = sk[t * ITEMS + r];
            val[r] = sv[t * ITEMS + r];
        }
        const uint32_t one = 1u << (16 * (t & 1));
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            const uint32_t d = (key[r] >> shift) & (kSmDigits - 1);
            if (t * ITEMS + r < A.n) atomicAdd(&cnt[d * (T / 2) + (t >> 1)], one);
        }
        __syncthreads();
        {
            const uint4 c0 = scan[0], c1 = scan[1];
            const uint32_t c[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
            uint32_t sum = 0;
#pragma unroll
            for (int q = 0; q < 8; ++q) sum += (c[q] & 0xFFFFu) + (c[q] >> 16);
            const uint32_t inc = wave_scan_dpp(sum);
            if (lane == 63) wsum[w] = inc;
            __syncthreads();
            // the waves' totals: lane v of every wave holds the total of waves 0..v
            const uint32_t tot = wave_scan_dpp(lane < T / 64 ? wsum[lane] : 0u);
            const uint32_t wbase = w == 0 ? 0u : (uint32_t)__builtin_amdgcn_readlane((int)tot, w - 1);
            uint32_t run = wbase + inc - sum;
            uint32_t o[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const uint32_t lo = run;
                run += c[q] & 0xFFFFu;
                o[q] = lo | (run << 16);
                run += c[q] >> 16;
            }
            scan[0] = make_uint4(o[0], o[1], o[2], o[3]);
            scan[1] = make_uint4(o[4], o[5], o[6], o[7]);
        }
        __syncthreads();
        // the LDS takes a wave's operations in order: equal digits of a thread
        // get their places in key order
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            const uint32_t d = (key[r] >> shift) & (kSmDigits - 1);
            pos[r] = 0;
            if (t * ITEMS + r < A.n)
                pos[r] = (atomicAdd(&cnt[d * (T / 2) + (t >> 1)], one) >> (16 * (t & 1))) & 0xFFFFu;
        }
#pragma unroll
        for (int r = 0; r < ITEMS; ++r)
            if (t * ITEMS + r < A.n) {   // pos: a permutation of 0..n-1
                sk[pos[r]] = key[r];
                sv[pos[r]] = val[r];
            }
        __syncthreads();
    }
    __syncthreads();
    for (int i = t; i < A.n; i += T) A.kout[i] = sk[i];
    for (int i = t; i < A.n; i += T) A.vout[i] = (int32_t)sv[i];
    if (!A.head) return;
    // bucket bounds: the last run start at or before a position, and the first
    // one after it, carried over the threads' consecutive positions by a scan
    // in each direction
    __shared__ int wlast[T / 64], wfirst[T / 64];
    uint16_t* sh = reinterpret_cast<uint16_t*>(cnt);   // heads, then (after them) ends: at most 4 T ITEMS bytes
    uint16_t* se = sh + T * ITEMS;
    const int i0 = t * ITEMS;
    uint32_t starts = 0;   // bit r: position i0 + r starts a run (or is the end)
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int i = i0 + r;
        const bool st = i == A.n || (i < A.n && (i == 0 || sk[i - 1] != sk[i]));
        starts |= st ? 1u << r : 0u;
    }
    int last = starts ? i0 + 31 - __builtin_clz(starts) : -1;
    int first = starts ? i0 + __builtin_ctz(starts) : 0x7FFFFFFF;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int u = __shfl_up(last, d, 64), v = __shfl_down(first, d, 64);
        if (lane >= d) last = max(last, u);
        if (lane + d < 64) first = min(first, v);
    }
    if (lane == 63) wlast[w] = last;
    if (lane == 0) wfirst[w] = first;
    __syncthreads();   // (sk is read: it takes the ranks)
    int before = __shfl_up(last, 1, 64), after = __shfl_down(first, 1, 64);   // of the threads before and after
    if (lane == 0) before = -1;
    if (lane == 63) after = A.n;
#pragma unroll
    for (int v = 0; v < T / 64; ++v) {
        if (v < w) before = max(before, wlast[v]);
        if (v > w) after = min(after, wfirst[v]);
    }
    after = min(after, A.n);
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int i = i0 + r;
        if (i < A.n) {
            const uint32_t lo = starts & (0xFFFFFFFFu >> (31 - r)), hi = starts >> (r + 1) << (r + 1);
            sh[i] = (uint16_t)(lo ? i0 + 31 - __builtin_clz(lo) : before);
            se[i] = (uint16_t)(hi ? i0 + __builtin_ctz(hi) : after);
            sk[sv[i]] = (uint32_t)i;
        }
    }
    __syncthreads();
    for (int i = t; i < A.n; i += T) {
        A.head[i] = (int32_t)sh[i];
        A.end[i] = (int32_t)se[i];
        A.rank[i] = (int32_t)sk[i];
    }
}

template <int ITEMS, int T = kSmThreads>
__global__ __launch_bounds__(T) void k_sort_small(SmSortArgs A) {
    mp_write_stamp(A.stamp);
    sort_small<ITEMS, T>(A);
}

template <int ITEMS, int T = kSmThreads>
__global__ __launch_bounds__(T) void k_sort_small_many(Many<SmSortArgs> M) {
    int block;
    const SmSortArgs A = many_args(M, block);
    sort_small<ITEMS, T>(A);
}

int64_t os_tiles(int64_t n) { return (n + kOsTile - 1) / kOsTile; }

int os_hist_blocks(int64_t n) {
    const int64_t per = (int64_t)kOsHistThreads * kOsHistKeys;
    return (int)std::max<int64_t>(1, std::min<int64_t>(kOsMaxHistBlocks, (n + per - 1) / per));
}

// Bits per pass and passes.  Wider digits where they save a pass: of 9 bits at
// any size (18-bit keys, hist and passes: 16,384 35 -> 24 us, 1,048,576 68 -> 51;
// 27 bits 43 -> 33 and 87 -> 75), of 10 only for up to two passes over few keys
// (20 bits: 16,384 34 -> 29 us, 65,536 35 -> 34, 262,144 46 -> 46, 1,048,576
// 68 -> 80; three such passes, 30 bits: 16,384 42 -> 42, 65,536 46 -> 49).
constexpr int64_t kOsWideMax = 32768;
struct OsPlan {
    int bits, passes;
};

OsPlan os_plan(int64_t n, int bits) {
    const auto passes = [&](int b) { return (bits + b - 1) / b; };
    if (passes(9) < passes(8)) return {9, passes(9)};
    if (passes(10) < passes(8) && passes(10) <= 2 && n <= kOsWideMax) return {10, passes(10)};
    return {8, std::min(kOsMaxPasses, passes(8))};
}

size_t os_scratch_words(int64_t n) {
    return (size_t)kOsHead + (size_t)os_tiles(n) * kOsMaxCounts + (size_t)kOsMaxHistBlocks * kOsMaxCounts;
}

// Stable sort of 32-bit keys by their low `bits` bits (one launch for the
// digit counts, one per pass), ping-ponging with the alt arrays; the
// result lands as in radix_sort.
void onesweep_sort(uint32_t* keys, int32_t* vals, uint32_t* keys_alt, int32_t* vals_alt, int64_t n, int bits,
                   DevMem& scratch, hipStream_t s, bool copy_back, uint64_t* stamp = nullptr) {
    if (n <= 1 || bits <= 0) return;
    if (n > (int64_t)kStVal) mp_throw(MP_E_UNSUPPORTED, "radix sort of more than 2^30 - 1 keys");
    const OsPlan plan = os_plan(n, bits);
    const int passes = plan.passes, digits = 1 << plan.bits;
    const int64_t tiles = os_tiles(n);
    const int nhist = os_hist_blocks(n);
    scratch.ensure(sizeof(uint32_t) * os_scratch_words(n));
    uint32_t* base = scratch.as<uint32_t>();
    uint32_t* status = base + kOsHead;
    uint32_t* part = status + (size_t)tiles * kOsMaxCounts;
    OsHistArgs H;
    H.keys = keys;
    H.n = n;
    H.passes = passes;
    H.bits = plan.bits;
    H.vec = ((uintptr_t)keys & 15u) == 0 ? 1 : 0;
    H.part = part;
    H.clear = base;
    H.clear_words = kOsHead + (int64_t)passes * tiles * digits;
    H.stamp = stamp;
    k_os_hist<<<nhist, kOsHistThreads, 0, s>>>(H);
    MP_CHECK_LAUNCH();
    uint32_t* ka = keys;
    int32_t* va = vals;
    uint32_t* kb = keys_alt;
    int32_t* vb = vals_alt;
    for (int p = 0; p < passes; ++p) {
        OsScatterArgs A;
        A.kin = ka;
        A.vin = va;
        A.kout = kb;
        A.vout = vb;
        A.n = n;
        A.shift = plan.bits * p;
        A.pass = p;
        A.nhist = nhist;
        A.part = part;
        A.status = status + (size_t)p * (size_t)tiles * digits;
        A.ticket = base + p;
        A.wait_flag = base + 4;
        if (plan.bits == 8) k_os_scatter<8><<<(unsigned)tiles, kOsThreads, 0, s>>>(A);
        else if (plan.bits == 9) k_os_scatter<9><<<(unsigned)tiles, kOsThreads, 0, s>>>(A);
        else k_os_scatter<10><<<(unsigned)tiles, kOsThreads, 0, s>>>(A);
        MP_CHECK_LAUNCH();
        std::swap(ka, kb);
        std::swap(va, vb);
    }
    if (copy_back && ka != keys) {
        MP_HIP(hipMemcpyAsync(keys, ka, sizeof(uint32_t) * (size_t)n, hipMemcpyDeviceToDevice, s));
        MP_HIP(hipMemcpyAsync(vals, va, sizeof(int32_t) * (size_t)n, hipMemcpyDeviceToDevice, s));
    }
}

}  // namespace

void mp_scan_exclusive_u32(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* total_dev, DevMem& scratch,
                           hipStream_t s) {
    scratch.ensure(sizeof(uint32_t) * (scan_scratch_words(n) + 16));
    scan_rec(in, out, n, total_dev, scratch.as<uint32_t>(), s);
}

size_t mp_radix_scratch_bytes(int64_t n) { return sizeof(uint32_t) * os_scratch_words(n); }

void mp_radix_sort_u32(uint32_t* keys, int32_t* vals, uint32_t* keys_alt, int32_t* vals_alt, int64_t n, int bits,
                       DevMem& scratch, hipStream_t s) {
    onesweep_sort(keys, vals, keys_alt, vals_alt, n, bits, scratch, s, true);
}

int mp_radix_passes(int64_t n, int bits) {
    return (n <= 1 || bits <= 0) ? 0 : os_plan(n, bits).passes;
}

void mp_radix_sort_u32_inplace_parity(uint32_t* keys, int32_t* vals, uint32_t* keys_alt, int32_t* vals_alt, int64_t n,
                                      int bits, DevMem& scratch, hipStream_t s, uint64_t* stamp) {
    onesweep_sort(keys, vals, keys_alt, vals_alt, n, bits, scratch, s, false, stamp);
}

bool mp_sort_is_small(int64_t n) { return n <= kSmMax; }

void mp_sort_small(const SmSortArgs& A, hipStream_t s) {
    // fewer waves wait less at the barriers: 16-bit keys, 1000 of them 10.1 us
    // with 1024 threads and 7.5 with 512, 2000 10.9 and 9.4, 4000 (8 a thread)
    // 12.9 and 14.1
    constexpr int kHalf = kSmThreads / 2;
    if (A.n <= 2 * kHalf) k_sort_small<2, kHalf><<<1, kHalf, 0, s>>>(A);
    else if (A.n <= 4 * kHalf) k_sort_small<4, kHalf><<<1, kHalf, 0, s>>>(A);
    else if (A.n <= kSmThreads * 4) k_sort_small<4><<<1, kSmThreads, 0, s>>>(A);
    else k_sort_small<kSmItems><<<1, kSmThreads, 0, s>>>(A);
    MP_CHECK_LAUNCH();
}

// (all with the layout of the largest)
void mp_sort_small_many(const std::vector<SmSortArgs>& a, ManyTab& T, hipStream_t s) {
    int n = 0;
    for (const SmSortArgs& A : a) n = std::max(n, A.n);
    constexpr int kHalf = kSmThreads / 2;
    unsigned grid;
    const Many<SmSortArgs> M = many_table(T, a, std::vector<int32_t>(a.size(), 1), grid);
    if (n <= 2 * kHalf) k_sort_small_many<2, kHalf><<<grid, kHalf, 0, s>>>(M);
    else if (n <= 4 * kHalf) k_sort_small_many<4, kHalf><<<grid, kHalf, 0, s>>>(M);
    else if (n <= kSmThreads * 4) k_sort_small_many<4><<<grid, kSmThreads, 0, s>>>(M);
    else k_sort_small_many<kSmItems><<<grid, kSmThreads, 0, s>>>(M);
    MP_CHECK_LAUNCH();
}

uint32_t* mp_radix_wait_flag(DevMem& scratch) { return scratch.as<uint32_t>() + 4; }

void mp_radix_sort_u64(uint64_t* keys, int32_t* vals, uint64_t* keys_alt, int32_t* vals_alt, int64_t n, int bits,
                       DevMem& scratch, hipStream_t s) {
    radix_sort<uint64_t>(keys, vals, keys_alt, vals_alt, n, bits, scratch, s);
}
