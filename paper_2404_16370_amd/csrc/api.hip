// api.hip -- the C-ABI of libmegapf: argument validation, handle lifetime,
// host/device pointer staging, the filter-step schedule and diagnostics.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <numeric>
#include <cstdio>
#include <cstring>
#include <memory>
#include <string>
#include <vector>

#include "megapf.h"
#include "mp_internal.hpp"
#include "mp_lsh.hpp"
#include "mp_place.hpp"

// ------------------------------------------------------------ errors
static thread_local std::string g_err;

void mp_throw(mp_status code, const char* fmt, ...) {
    char buf[1024];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    throw MpError{code, std::string(buf)};
}

template <class F>
static mp_status guarded(const char* where, F&& fn) {
    try {
        fn();
        return MP_OK;
    } catch (const MpError& e) {
        g_err = std::string(where) + ": " + e.msg;
        return e.code;
    } catch (const std::exception& e) {
        g_err = std::string(where) + ": " + e.what();
        return MP_E_HIP;
    }
}

extern "C" const char* mp_last_error(void) { return g_err.c_str(); }

// error handling of the other translation units' entry points
mp_status mp_guarded_call(const char* where, void (*fn)(void*), void* ctx) {
    return guarded(where, [&]() { fn(ctx); });
}

// ------------------------------------------------------------ device memory
void DevMem::alloc(size_t b) {
    release();
    if (b == 0) b = 16;
    const hipError_t e = hipMalloc(&p, b);
    if (e != hipSuccess) {
        p = nullptr;
        (void)hipGetLastError();
        mp_throw(e == hipErrorOutOfMemory ? MP_E_OOM : MP_E_HIP, "hipMalloc(%zu): %s", b, hipGetErrorString(e));
    }
    bytes = b;
}
void DevMem::ensure(size_t b) {
    if (bytes < b) alloc(b);
}
void DevMem::part_of(const DevMem& whole, size_t offset, size_t b) {
    release();
    p = whole.as<char>() + offset;
    bytes = b;
    part = true;
}
void DevMem::release() {
    if (p && !part) (void)hipFree(p);
    p = nullptr;
    bytes = 0;
    part = false;
}

const void* ManyTab::put(const void* data, size_t n) {
    const size_t at = (host.size() + 15) / 16 * 16;
    if (at + n > dev.bytes) mp_throw(MP_E_STATE, "launch tables of %zu bytes are full", dev.bytes);
    host.resize(at + n);
    std::memcpy(host.data() + at, data, n);
    return dev.as<char>() + at;
}

constexpr size_t kStampMarks = 2;   // clock values of a scan upload before those of a step

void HostMem::ensure(size_t b) {
    if (bytes >= b) return;
    if (p) (void)hipHostFree(p);
    p = nullptr;
    bytes = 0;
    const hipError_t e = hipHostMalloc(&p, b, hipHostMallocDefault);
    if (e != hipSuccess) {
        p = nullptr;
        (void)hipGetLastError();
        mp_throw(e == hipErrorOutOfMemory ? MP_E_OOM : MP_E_HIP, "hipHostMalloc(%zu): %s", b, hipGetErrorString(e));
    }
    bytes = b;
}

static inline hipStream_t as_stream(void* s) { return static_cast<hipStream_t>(s); }

// false: memory that the runtime does not know (ordinary host memory)
static bool pointer_attr(const void* p, hipPointerAttribute_t& a) {
    std::memset(&a, 0, sizeof(a));
    const hipError_t e = hipPointerGetAttributes(&a, p);
    if (e != hipSuccess) (void)hipGetLastError();
    return e == hipSuccess;
}

static bool is_device_ptr(const void* p) {
    hipPointerAttribute_t a;
    return pointer_attr(p, a) && (a.type == hipMemoryTypeDevice || a.type == hipMemoryTypeManaged);
}

// bring `bytes` of caller data into device memory (no copy for device pointers)
static const void* stage_in(const void* src, size_t bytes, DevMem& tmp, hipStream_t s) {
    if (bytes == 0) return nullptr;
    if (is_device_ptr(src)) return src;
    tmp.ensure(bytes);
    MP_HIP(hipMemcpyAsync(tmp.p, src, bytes, hipMemcpyHostToDevice, s));
    return tmp.p;
}

// copy caller data to host memory (for validation)
static void fetch_host(const void* src, size_t bytes, void* dst, hipStream_t s) {
    if (bytes == 0) return;
    if (is_device_ptr(src)) {
        MP_HIP(hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, s));
        MP_HIP(hipStreamSynchronize(s));
    } else {
        std::memcpy(dst, src, bytes);
    }
}

static void copy_out(void* dst, const void* src_dev, size_t bytes, hipStream_t s) {
    if (bytes == 0) return;
    MP_HIP(hipMemcpyAsync(dst, src_dev, bytes, hipMemcpyDefault, s));
    if (!is_device_ptr(dst)) MP_HIP(hipStreamSynchronize(s));
}

static bool all_finite(const float* p, size_t n) {
    for (size_t i = 0; i < n; ++i)
        if (!std::isfinite(p[i])) return false;
    return true;
}

// ------------------------------------------------------------ map
extern "C" void mp_map_default_params(mp_map_params* p) {
    if (!p) return;
    p->voxel = 0.5f;
    p->nnf_radius = 2;
    p->min_points = 5;
    p->cov_eps = 1e-3f;
    p->backend = MP_NNF_AUTO;
    p->gauss_mode = MP_GAUSS_VOXEL;
    p->point_k = 10;
    p->point_search = 2;
}

extern "C" mp_status mp_map_build(const float* xyz, int64_t n, const mp_map_params* params, void* stream,
                                  mp_map* out) {
    return guarded("mp_map_build", [&]() {
        if (!out || !params || n < 0 || (n > 0 && !xyz)) mp_throw(MP_E_ARG, "null argument or n < 0");
        if (!(params->voxel > 0.0f) || !std::isfinite(params->voxel)) mp_throw(MP_E_ARG, "voxel must be > 0");
        if (params->nnf_radius < 0 || params->nnf_radius > 8) mp_throw(MP_E_ARG, "nnf_radius must be 0..8");
        if (params->min_points < 3) mp_throw(MP_E_ARG, "min_points must be >= 3");
        if (!(params->cov_eps > 0.0f && params->cov_eps <= 1.0f)) mp_throw(MP_E_ARG, "cov_eps must be in (0, 1]");
        if (params->backend < MP_NNF_AUTO || params->backend > MP_NNF_DENSE) mp_throw(MP_E_ARG, "bad backend");
        if (params->gauss_mode != MP_GAUSS_VOXEL && params->gauss_mode != MP_GAUSS_POINT)
            mp_throw(MP_E_ARG, "bad gauss_mode");
        if (params->gauss_mode == MP_GAUSS_POINT) {
            if (params->point_k < 3 || params->point_k > 32) mp_throw(MP_E_ARG, "point_k must be 3..32");
            if (params->point_search < 1 || params->point_search > 4) mp_throw(MP_E_ARG, "point_search must be 1..4");
            if (params->nnf_radius < 1)
                mp_throw(MP_E_ARG, "per-point Gaussians need nnf_radius >= 1 (the field reaches nnf_radius * voxel)");
            if (params->backend == MP_NNF_HASH)
                mp_throw(MP_E_UNSUPPORTED, "per-point Gaussians take the dense field only");
        }
        if (n > (int64_t)INT32_MAX) mp_throw(MP_E_UNSUPPORTED, "more than 2^31-1 map points");
        hipStream_t s = as_stream(stream);
        mp_map m = new mp_map_s();
        m->params = *params;
        try {
            DevMem tmp;
            const float* d = static_cast<const float*>(stage_in(xyz, sizeof(float) * 3 * (size_t)n, tmp, s));
            mp_build_map(m, d, n, s);
            MP_HIP(hipStreamSynchronize(s));
        } catch (...) {
            delete m;
            throw;
        }
        *out = m;
    });
}

extern "C" mp_status mp_debug_map_point_knn(const float* xyz, int64_t n, const mp_map_params* params,
                                            int32_t* knn_out, void* stream) {
    return guarded("mp_debug_map_point_knn", [&]() {
        if (!params || !knn_out || n <= 0 || !xyz) mp_throw(MP_E_ARG, "null argument or n <= 0");
        if (params->gauss_mode != MP_GAUSS_POINT) mp_throw(MP_E_ARG, "gauss_mode must be POINT");
        if (params->point_k < 3 || params->point_k > 32) mp_throw(MP_E_ARG, "point_k must be 3..32");
        if (n > (int64_t)INT32_MAX) mp_throw(MP_E_UNSUPPORTED, "more than 2^31-1 map points");
        hipStream_t s = as_stream(stream);
        const size_t bytes = sizeof(int32_t) * (size_t)n * (size_t)params->point_k;
        DevMem lists;
        lists.alloc(bytes);
        mp_map m = new mp_map_s();
        m->params = *params;
        m->knn_dbg = lists.as<int32_t>();
        try {
            DevMem tmp;
            const float* d = static_cast<const float*>(stage_in(xyz, sizeof(float) * 3 * (size_t)n, tmp, s));
            mp_build_map(m, d, n, s);
            MP_HIP(hipMemcpyAsync(knn_out, lists.p, bytes, hipMemcpyDefault, s));
            MP_HIP(hipStreamSynchronize(s));
        } catch (...) {
            delete m;
            throw;
        }
        delete m;
    });
}

namespace {
__global__ void k_iota(int32_t* v, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) v[i] = (int32_t)i;
}
}  // namespace

extern "C" mp_status mp_debug_sort_u32(const uint32_t* keys, int64_t n, int32_t bits, uint32_t* keys_out,
                                       int32_t* order_out, void* stream) {
    return guarded("mp_debug_sort_u32", [&]() {
        if (!keys || !keys_out || !order_out || n <= 0) mp_throw(MP_E_ARG, "null argument or n <= 0");
        if (bits < 1 || bits > 32) mp_throw(MP_E_ARG, "bits must be 1..32");
        if (n >= ((int64_t)1 << 30)) mp_throw(MP_E_UNSUPPORTED, "2^30 or more keys");
        hipStream_t s = as_stream(stream);
        DevMem k, k2, v, v2, scratch;
        k.alloc(sizeof(uint32_t) * (size_t)n);
        k2.alloc(sizeof(uint32_t) * (size_t)n);
        v.alloc(sizeof(int32_t) * (size_t)n);
        v2.alloc(sizeof(int32_t) * (size_t)n);
        scratch.alloc(mp_radix_scratch_bytes(n));
        mp_fill_u32(mp_radix_wait_flag(scratch), 0u, 1, s);
        MP_HIP(hipMemcpyAsync(k.p, keys, sizeof(uint32_t) * (size_t)n, hipMemcpyDefault, s));
        k_iota<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(v.as<int32_t>(), n);
        MP_CHECK_LAUNCH();
        mp_radix_sort_u32(k.as<uint32_t>(), v.as<int32_t>(), k2.as<uint32_t>(), v2.as<int32_t>(), n, bits, scratch, s);
        uint32_t waited = 0;
        MP_HIP(hipMemcpyAsync(keys_out, k.p, sizeof(uint32_t) * (size_t)n, hipMemcpyDefault, s));
        MP_HIP(hipMemcpyAsync(order_out, v.p, sizeof(int32_t) * (size_t)n, hipMemcpyDefault, s));
        MP_HIP(hipMemcpyAsync(&waited, mp_radix_wait_flag(scratch), 4, hipMemcpyDeviceToHost, s));
        MP_HIP(hipStreamSynchronize(s));
        if (waited == 1) mp_throw(MP_E_HIP, "a sort workgroup stopped waiting for its predecessors' digit counts");
        if (waited) mp_throw(MP_E_HIP, "a key's sorted place fell outside the output");
    });
}

extern "C" mp_status mp_map_get_info(mp_map map, mp_map_info* out) {
    return guarded("mp_map_get_info", [&]() {
        if (!map || !out) mp_throw(MP_E_ARG, "null argument");
        *out = map->info;
    });
}

extern "C" mp_status mp_map_get_gauss(mp_map map, float* mu, float* normal, int32_t* voxel, int32_t* count,
                                      void* stream) {
    return guarded("mp_map_get_gauss", [&]() {
        if (!map) mp_throw(MP_E_ARG, "null map");
        const int64_t G = map->info.num_gauss;
        if (G == 0) return;
        hipStream_t s = as_stream(stream);
        std::vector<float4> g((size_t)(2 * G));
        MP_HIP(hipMemcpyAsync(g.data(), map->gauss.p, sizeof(float4) * 2 * G, hipMemcpyDeviceToHost, s));
        MP_HIP(hipStreamSynchronize(s));
        std::vector<float> hm(3 * G), hn(3 * G);
        std::vector<int32_t> hv(3 * G), hc(G);
        MP_HIP(hipMemcpyAsync(hv.data(), map->vox.p, sizeof(int32_t) * 3 * G, hipMemcpyDeviceToHost, s));
        MP_HIP(hipStreamSynchronize(s));
        for (int64_t k = 0; k < G; ++k) {
            hm[3 * k] = g[2 * k].x; hm[3 * k + 1] = g[2 * k].y; hm[3 * k + 2] = g[2 * k].z;
            hc[k] = (int32_t)g[2 * k].w;
            hn[3 * k] = g[2 * k + 1].x; hn[3 * k + 1] = g[2 * k + 1].y; hn[3 * k + 2] = g[2 * k + 1].z;
        }
        if (mu) copy_out(mu, hm.data(), sizeof(float) * 3 * G, s);
        if (normal) copy_out(normal, hn.data(), sizeof(float) * 3 * G, s);
        if (voxel) copy_out(voxel, hv.data(), sizeof(int32_t) * 3 * G, s);
        if (count) copy_out(count, hc.data(), sizeof(int32_t) * G, s);
        MP_HIP(hipStreamSynchronize(s));
    });
}

extern "C" mp_status mp_map_lookup(mp_map map, const float* xyz, int64_t n, int32_t* gid_out, void* stream) {
    return guarded("mp_map_lookup", [&]() {
        if (!map || n < 0 || (n > 0 && (!xyz || !gid_out))) mp_throw(MP_E_ARG, "null argument or n < 0");
        if (n == 0) return;
        hipStream_t s = as_stream(stream);
        DevMem tin, tout;
        const float* d = static_cast<const float*>(stage_in(xyz, sizeof(float) * 3 * (size_t)n, tin, s));
        if (map->info.num_gauss == 0) {
            std::vector<int32_t> miss((size_t)n, -1);
            copy_out(gid_out, miss.data(), sizeof(int32_t) * n, s);
            MP_HIP(hipStreamSynchronize(s));
            return;
        }
        int32_t* o = gid_out;
        const bool dev_out = is_device_ptr(gid_out);
        if (!dev_out) {
            tout.alloc(sizeof(int32_t) * (size_t)n);
            o = tout.as<int32_t>();
        }
        mp_map_lookup_launch(map->view, d, n, o, s);
        if (!dev_out) copy_out(gid_out, o, sizeof(int32_t) * n, s);
    });
}

extern "C" mp_status mp_map_destroy(mp_map map) {
    return guarded("mp_map_destroy", [&]() {
        if (!map) return;
        if (map->users > 0) mp_throw(MP_E_STATE, "map still used by %d filter(s)", map->users);
        MP_HIP(hipDeviceSynchronize());
        delete map;
    });
}

// ------------------------------------------------------------ filter
extern "C" void mp_filter_default_params(mp_filter_params* p) {
    if (!p) return;
    std::memset(p, 0, sizeof(*p));
    p->n_particles = 4096;
    p->k = 16;
    p->lsh_bits = 20;
    p->svgd_iters = 10;
    p->post_iters = 10;
    p->window_c = 32;
    p->scan_k = 10;
    p->sigma_r = 5.0f;
    p->sigma_t = 2.5f;
    p->lsh_alpha = 1.0f;
    p->lsh_sigma = 0.3f;
    p->c_max = 9.0f;
    p->d_max = 1.0f;
    p->lambda_rel = 1e-3f;
    p->lambda_abs = 1e-6f;
    p->temperature = 1.0f;
    p->prior_floor = 1e-30f;
    p->cov_eps = 1e-3f;
    p->lik_chunks = 0;
    p->lik_batch = 0;
    p->scorer = MP_SCORER_PLAIN;
    p->sigma_s = 0.03f;
    p->lsh_tangent = MP_LSH_TANGENT_DECOUPLED;
    p->lsh_tables = 1;
    p->svgd_grad = MP_SVGD_GRAD_APPROX;
    p->svgd_transport = MP_SVGD_TRANSPORT_NONE;
    p->final_rescore = 0;
    p->seed = 1;
}

static void validate_params(const mp_filter_params& p) {
    if (p.n_particles < 1 || p.n_particles > (1 << 26)) mp_throw(MP_E_ARG, "n_particles must be 1..2^26");
    if (p.k < 1 || p.k > 32) mp_throw(MP_E_ARG, "k must be 1..32");
    if (p.lsh_bits < 0 || p.lsh_bits > 30) mp_throw(MP_E_ARG, "lsh_bits must be 0..30");
    if (p.svgd_iters < 0 || p.post_iters < 0 || p.window_c < 0) mp_throw(MP_E_ARG, "negative iteration count");
    if (p.scan_k < 3 || p.scan_k > 32) mp_throw(MP_E_ARG, "scan_k must be 3..32");
    const float fs[] = {p.sigma_r, p.sigma_t, p.lsh_alpha, p.lsh_sigma, p.c_max, p.d_max,
                        p.lambda_rel, p.lambda_abs, p.temperature, p.prior_floor, p.cov_eps};
    for (float v : fs)
        if (!std::isfinite(v)) mp_throw(MP_E_ARG, "non-finite parameter");
    if (p.sigma_r < 0 || p.sigma_t < 0 || p.lsh_alpha <= 0 || p.lsh_sigma < 0 || p.c_max <= 0 || p.d_max <= 0 ||
        p.lambda_rel < 0 || p.lambda_abs < 0 || p.temperature <= 0 || p.prior_floor < 0 || p.cov_eps <= 0 ||
        p.cov_eps > 1)
        mp_throw(MP_E_ARG, "parameter out of range");
    if (p.lik_chunks < 0) mp_throw(MP_E_ARG, "lik_chunks must be >= 0");
    if (p.lik_batch != 0 && p.lik_batch != 1 && p.lik_batch != 2 && p.lik_batch != 4 && p.lik_batch != 8 &&
        p.lik_batch != 16 && p.lik_batch != 32)
        mp_throw(MP_E_ARG, "lik_batch must be 0, 1, 2, 4, 8, 16 or 32");
    if (p.scorer < MP_SCORER_PLAIN || p.scorer > MP_SCORER_SURROGATE) mp_throw(MP_E_ARG, "unknown scorer");
    if (p.lik_layout < MP_LIK_LAYOUT_AUTO || p.lik_layout > MP_LIK_LAYOUT_GROUPED) mp_throw(MP_E_ARG, "unknown lik_layout");
    if (!std::isfinite(p.sigma_s) || !(p.sigma_s > 0.0f)) mp_throw(MP_E_ARG, "sigma_s must be positive");
    if (p.lsh_tangent != MP_LSH_TANGENT_DECOUPLED && p.lsh_tangent != MP_LSH_TANGENT_SE3)
        mp_throw(MP_E_ARG, "unknown lsh_tangent");
    if (p.lsh_tables < 0 || p.lsh_tables > 16) mp_throw(MP_E_ARG, "lsh_tables must be 0..16");
    if (p.svgd_grad != MP_SVGD_GRAD_APPROX && p.svgd_grad != MP_SVGD_GRAD_EXACT) mp_throw(MP_E_ARG, "unknown svgd_grad");
    if (p.svgd_transport != MP_SVGD_TRANSPORT_NONE && p.svgd_transport != MP_SVGD_TRANSPORT_ADJOINT)
        mp_throw(MP_E_ARG, "unknown svgd_transport");
    if (p.final_rescore != 0 && p.final_rescore != 1) mp_throw(MP_E_ARG, "final_rescore must be 0 or 1");
}

static void destroy_filter(mp_filter f) {
    if (!f) return;
    if (f->map) f->map->users--;
    if (f->sur) f->sur->users--;
    if (f->step_ev) (void)hipEventDestroy(f->step_ev);
    if (f->scan_ev) (void)hipEventDestroy(f->scan_ev);
    delete f;
}

extern "C" mp_status mp_filter_init(mp_map map, const mp_filter_params* params, const mp_init_desc* init,
                                    void* stream, mp_filter* out) {
    return guarded("mp_filter_init", [&]() {
        if (!map || !params || !init || !out) mp_throw(MP_E_ARG, "null argument");
        validate_params(*params);
        const int n = params->n_particles;
        hipStream_t s = as_stream(stream);
        std::vector<float> host_poses;
        float gmean[7], gL[36];
        bool gnoise = false;
        if (init->kind == MP_INIT_EXPLICIT) {
            if (!init->poses) mp_throw(MP_E_ARG, "explicit init without poses");
            std::vector<float> p7((size_t)n * 7);
            fetch_host(init->poses, sizeof(float) * 7 * (size_t)n, p7.data(), s);
            if (!all_finite(p7.data(), p7.size())) mp_throw(MP_E_ARG, "non-finite initial pose");
            host_poses.assign((size_t)n * 8, 0.0f);
            for (int i = 0; i < n; ++i) {
                const float* q = &p7[7 * (size_t)i];
                const double nq = std::sqrt((double)q[0] * q[0] + (double)q[1] * q[1] + (double)q[2] * q[2] +
                                            (double)q[3] * q[3]);
                if (!(nq > 1e-12)) mp_throw(MP_E_ARG, "zero quaternion for particle %d", i);
                const bool unit = std::fabs(nq - 1.0) < 1e-6;
                for (int k = 0; k < 4; ++k) host_poses[8 * (size_t)i + k] = unit ? q[k] : (float)(q[k] / nq);
                for (int k = 0; k < 3; ++k) host_poses[8 * (size_t)i + 4 + k] = q[4 + k];
            }
        } else if (init->kind == MP_INIT_UNIFORM_BOX) {
            if (!all_finite(init->box_min, 3) || !all_finite(init->box_max, 3)) mp_throw(MP_E_ARG, "non-finite box");
            for (int a = 0; a < 3; ++a)
                if (init->box_max[a] < init->box_min[a]) mp_throw(MP_E_ARG, "box_max < box_min");
        } else if (init->kind == MP_INIT_GAUSSIAN) {
            // the mean replicated, then moved by exp(L z_i) as a prediction from it would be
            mp_prepare_prediction(init->mean, init->cov, gmean, gL, gnoise);
            host_poses.assign((size_t)n * 8, 0.0f);
            for (int i = 0; i < n; ++i)
                for (int k = 0; k < 7; ++k) host_poses[8 * (size_t)i + k] = gmean[k];
        } else {
            mp_throw(MP_E_ARG, "unknown init kind %d", init->kind);
        }
        mp_filter f = new mp_filter_s();
        try {
            MP_HIP(hipGetDevice(&f->device));
            f->map = map;
            map->users++;
            f->p = *params;
            f->n = n;
            f->K = params->k;
            for (int a = 0; a < 3; ++a) {
                f->lsh_lo[a] = map->box_lo[a];
                f->lsh_hi[a] = map->box_hi[a];
            }
            const size_t N = (size_t)n, K = (size_t)params->k;
            // one clock value per mark of a step: prediction, re-score, posterior, end; per iteration
            // three list stages per table, three of the likelihood, SVGD (stages beyond 2^16 iterations' marks
            // are not timed)
            const size_t per = 3 * (size_t)std::max(1, params->lsh_tables) + 4;
            // One allocation for all of them: a call each, for allocating and for
            // freeing, took 0.7 and 4.8 ms for a filter of 1,048,576 particles, 0.13
            // and 0.6 ms now.
            const struct {
                DevMem* m;
                size_t bytes;
            } parts[] = {
                {&f->poses[0], 32 * N},
                {&f->poses[1], 32 * N},
                {&f->psi, 32 * N},
                {&f->codes, 4 * N},
                {&f->sorted, 4 * N},
                {&f->scodes, 4 * N},
                {&f->tmp_keys, 4 * N},
                {&f->tmp_vals, 4 * N},
                {&f->lkeys, 4 * N},
                {&f->lorder, 4 * N},
                {&f->head, 4 * N},
                {&f->end, 4 * N},
                {&f->rank, 4 * N},
                {&f->hist, mp_radix_scratch_bytes(n)},
                {&f->nbr, 4 * K * N},
                {&f->kval, 4 * K * N},
                {&f->cnt, 4 * N},
                {&f->prior, 4 * N},
                {&f->post0, 4 * N},
                {&f->post1, 4 * N},
                {&f->flags, 64},
                {&f->tlsh, 32},
                {&f->stamps, sizeof(uint64_t) *
                                 (kStampMarks + 8 + per * (size_t)std::min(params->svgd_iters, 1 << 16))},
                {&f->stepinfo, 16 * sizeof(double)},
                {&f->red, sizeof(double) * (N + 3 * ((N + 255) / 256)) + sizeof(int) * ((N + 255) / 256) + 64},
            };
            const auto padded = [](size_t b) { return (b + 255) / 256 * 256; };
            size_t total = 0;
            for (const auto& q : parts) total += padded(q.bytes);
            f->arena.alloc(total);
            size_t at = 0;
            for (const auto& q : parts) {
                q.m->part_of(f->arena, at, q.bytes);
                at += padded(q.bytes);
            }
            mp_fill_u32(mp_radix_wait_flag(f->hist), 0u, 1, s);   // (sorts in one workgroup leave it)
            MP_HIP(hipMemsetAsync(f->flags.p, 0, 64, s));
            MP_HIP(hipMemsetAsync(f->stepinfo.p, 0, 16 * sizeof(double), s));
            MP_HIP(hipMemsetAsync(f->psi.p, 0, 32 * N, s));
            MP_HIP(hipMemsetAsync(f->tlsh.p, 0, 32, s));
            MP_HIP(hipMemsetAsync(f->post1.p, 0, 4 * N, s));
            if (init->kind == MP_INIT_EXPLICIT || init->kind == MP_INIT_GAUSSIAN) {
                MP_HIP(hipMemcpyAsync(f->poses[0].p, host_poses.data(), 32 * N, hipMemcpyHostToDevice, s));
                if (init->kind == MP_INIT_GAUSSIAN) {
                    static const float ident[7] = {1, 0, 0, 0, 0, 0, 0};
                    mp_launch_predict(f, ident, gL, gnoise, s, true);
                }
                MP_HIP(hipStreamSynchronize(s));
            } else {
                mp_launch_init_uniform(f, init->box_min, init->box_max, s);
            }
            mp_launch_reset_lists(f, s);
        } catch (...) {
            destroy_filter(f);
            throw;
        }
        *out = f;
    });
}

extern "C" mp_status mp_filter_destroy(mp_filter f) {
    return guarded("mp_filter_destroy", [&]() {
        if (!f) return;
        if (f->batch_users > 0) mp_throw(MP_E_STATE, "filter still held by %d batch(es)", f->batch_users);
        MP_HIP(hipDeviceSynchronize());
        destroy_filter(f);
    });
}

// The verdict of a scan's check, 15 us after the call on an idle stream: polled
// for a while, as waiting for the stream costs as much again and would wait for
// the sort as well.  (An upload of 300 points returned after 42 us and was done
// after 85 with the verdict copied back before the sort; 20 and 50 us now.)
static uint32_t scan_verdict(const ScanPrep& P, hipStream_t s) {
    const auto read = [&]() { return __atomic_load_n(P.verdict, __ATOMIC_ACQUIRE); };
    const auto t0 = std::chrono::steady_clock::now();
    while (read() >> 2 != P.seq)
        if (std::chrono::steady_clock::now() - t0 > std::chrono::microseconds(200)) {   // behind other work
            MP_HIP(hipStreamSynchronize(s));
            if (read() >> 2 != P.seq) mp_throw(MP_E_HIP, "no verdict on the scan");
            break;
        }
    return read() & 3u;
}

// The clock values [from, from + count) to the host and an event behind them, for a
// filter whose stage times are asked for: mp_stage_times then waits for that
// event, and not for other work on the device.  (Not for every filter: the events
// alone, one with each upload and step, took a frame of 256 particles from 153 to
// 160 us.)
static bool leave_times(mp_filter f, hipEvent_t ev, size_t from, size_t count, hipStream_t s) {
    if (!ev || sizeof(uint64_t) * (from + count) > f->stamps.bytes) return false;
    MP_HIP(hipMemcpyAsync(f->times.as<uint64_t>() + from, f->stamps.as<uint64_t>() + from, sizeof(uint64_t) * count,
                          hipMemcpyDeviceToHost, s));
    MP_HIP(hipEventRecord(ev, s));
    return true;
}

extern "C" mp_status mp_scan_upload(mp_filter f, const float* xyz, const float* cov6, int32_t n, void* stream) {
    return guarded("mp_scan_upload", [&]() {
        if (!f || n < 0 || (n > 0 && !xyz)) mp_throw(MP_E_ARG, "null argument or n < 0");
        if (n > 65536) mp_throw(MP_E_ARG, "more than 65536 scan points");
        hipStream_t s = as_stream(stream);
        if (n > 0) {
            f->scan_xyz.ensure(sizeof(float) * 3 * (size_t)n);
            f->scan_perm.ensure(sizeof(int32_t) * (size_t)n);
            f->scan_work.ensure(sizeof(float4) * (2 * kPrepParts + 1) + sizeof(uint32_t) * 5 * (size_t)n);
            if (!f->scan_verdict.p) {
                f->scan_verdict.ensure(64);
                *f->scan_verdict.as<uint32_t>() = 0;   // the number of no scan
            }
            f->scan_sort.ensure(mp_radix_scratch_bytes(n));
            // caller data (host or device) into the filter's staging buffers
            MP_HIP(hipMemcpyAsync(f->scan_xyz.p, xyz, sizeof(float) * 3 * (size_t)n, hipMemcpyDefault, s));
            const float* dcov = nullptr;
            if (cov6) {
                f->scan_cov.ensure(sizeof(float) * 6 * (size_t)n);
                MP_HIP(hipMemcpyAsync(f->scan_cov.p, cov6, sizeof(float) * 6 * (size_t)n, hipMemcpyDefault, s));
                dcov = f->scan_cov.as<float>();
            }
            // Walk order for the likelihood: Morton order of the points on a grid of half the
            // map voxel, so that consecutive points of one particle land in the same or
            // neighbouring voxels (the sum over points does not depend on the order).
            // Only the verdict of the check comes back: the sort runs while the host waits for
            // it.  Nothing before it touches what a refused scan must leave alone.
            ScanPrep P;
            P.part = f->scan_work.as<float4>();
            P.start = reinterpret_cast<uint64_t*>(P.part + 2 * kPrepParts);
            P.key = reinterpret_cast<uint32_t*>(P.part + 2 * kPrepParts + 1);
            P.idx = f->scan_perm.as<int32_t>();
            P.xyz = f->scan_xyz.as<float>();
            P.cov = dcov;
            P.verdict = f->scan_verdict.as<uint32_t>();
            P.seq = f->scan_seq = f->scan_seq % 0x3FFFFFFFu + 1;
            P.n = n;
            uint32_t* key_alt = P.key + n;
            int32_t* work[3];   // an order's second buffer, the index's order, places in the walk order
            for (size_t k = 0; k < 3; ++k) work[k] = reinterpret_cast<int32_t*>(P.key + (2 + k) * (size_t)n);
            mp_scan_walk_order(P, 0.5f * f->map->params.voxel, key_alt, work[0], f->scan_sort, s);
            const uint32_t verdict = scan_verdict(P, s);
            if (verdict & 1u) {
                // (the sort: an upload that answers the refusal may come on another stream)
                MP_HIP(hipStreamSynchronize(s));
                mp_throw(MP_E_ARG, cov6 ? "non-finite scan point or covariance" : "non-finite scan point");
            }
            // The current records become the previous scan's (odometry), whose places take the
            // new ones.  Larger places are all there before an old one is given up, so that a
            // failed allocation leaves the last two scans as a refusal does.
            const bool follows = f->orig_n > 0;
            DevMem& orig = follows ? f->prev_orig : f->scan_orig;
            DevMem& idx = follows ? f->prev_idx : f->scan_idx;
            const size_t rec_bytes = sizeof(float) * 12 * (size_t)n, idx_bytes = mp_scan_index_bytes(n);
            bool own = (verdict & 2u) != 0;
            {
                DevMem walk_new, orig_new, idx_new, own_new;
                if (f->scan.bytes < rec_bytes) walk_new.alloc(rec_bytes);
                if (orig.bytes < rec_bytes) orig_new.alloc(rec_bytes);
                if (idx.bytes < idx_bytes) idx_new.alloc(idx_bytes);
                if (own && f->scan_own.bytes < rec_bytes) {
                    try {
                        own_new.alloc(rec_bytes);
                    } catch (const MpError&) {
                        own = false;   // no room: the index keeps the walk order
                    }
                }
                if (walk_new.p) f->scan.swap(walk_new);
                if (orig_new.p) orig.swap(orig_new);
                if (idx_new.p) idx.swap(idx_new);
                if (own_new.p) f->scan_own.swap(own_new);
            }
            if (follows) {
                f->scan_orig.swap(f->prev_orig);
                f->scan_idx.swap(f->prev_idx);
                f->prev_n = f->orig_n;
            }
            f->orig_n = n;
            f->idx_own = own;
            const int32_t* perm = P.idx;
            ScanRecords R{f->scan_orig.as<float4>(), f->scan.as<float4>(), nullptr, nullptr};
            if (f->idx_own) {
                mp_scan_index_order(P, key_alt, work[1], work[0], work[2], f->scan_sort, s);
                perm = work[1];
                R.index = f->scan_own.as<float4>();
                R.walk = f->scan.as<float4>();
                R.wpos = work[2];
            }
            mp_scan_records(P.xyz, dcov, perm, n, f->p.scan_k, f->p.cov_eps, mp_scan_index(f->scan_idx, n), R, P.start,
                            f->stamps.as<uint64_t>(), s);
            f->scan_timed = true;
            f->scan_rec = leave_times(f, f->scan_ev, 0, kStampMarks, s);
        }
        f->scan_n = n;
        f->last_stream = s;
    });
}

void mp_stage_begin(mp_filter f, int st) {
    if (!f->timing) return;
    uint64_t* base = f->stamps.as<uint64_t>();
    int32_t slot = kStampMarks + (int32_t)f->marks.size();
    if (sizeof(uint64_t) * ((size_t)slot + 2) > f->stamps.bytes) {   // (one slot is left for the end)
        f->timing = false;
        f->stamp = nullptr;
        return;
    }
    if (f->stamp) slot = f->marks.back().slot;   // the stage before launched nothing: both start here
    f->marks.push_back({st, slot});
    f->stamp = base + slot;
}

// host FP64 Cholesky of a 6x6 PSD matrix; false if not PSD
static bool chol6_host(const double A[36], double L[36]) {
    std::memset(L, 0, sizeof(double) * 36);
    double scale = 0.0;
    for (int i = 0; i < 6; ++i) scale = std::fmax(scale, std::fabs(A[7 * i]));
    const double tol = -1e-9 * (scale > 0 ? scale : 1.0);
    for (int j = 0; j < 6; ++j) {
        double s = A[6 * j + j];
        for (int k = 0; k < j; ++k) s -= L[6 * j + k] * L[6 * j + k];
        if (s < tol) return false;
        s = s > 0 ? s : 0.0;
        L[6 * j + j] = std::sqrt(s);
        for (int i = j + 1; i < 6; ++i) {
            double t = A[6 * i + j];
            for (int k = 0; k < j; ++k) t -= L[6 * i + k] * L[6 * j + k];
            L[6 * i + j] = L[6 * j + j] > 0 ? t / L[6 * j + j] : 0.0;
        }
    }
    return true;
}

void mp_prepare_prediction(const float dT[7], const float cov[36], float dq[7], float Lf[36], bool& noise) {
    if (!all_finite(dT, 7)) mp_throw(MP_E_ARG, "non-finite dT");
    const double nq = std::sqrt((double)dT[0] * dT[0] + (double)dT[1] * dT[1] + (double)dT[2] * dT[2] +
                                (double)dT[3] * dT[3]);
    if (!(nq > 1e-12)) mp_throw(MP_E_ARG, "zero quaternion in dT");
    for (int k = 0; k < 4; ++k) dq[k] = (float)(dT[k] / nq);
    for (int k = 0; k < 3; ++k) dq[4 + k] = dT[4 + k];
    noise = false;
    std::memset(Lf, 0, sizeof(float) * 36);
    if (cov) {
        if (!all_finite(cov, 36)) mp_throw(MP_E_ARG, "non-finite cov_dT");
        double A[36], L[36];
        for (int i = 0; i < 6; ++i)
            for (int j = 0; j < 6; ++j) {
                if (std::fabs((double)cov[6 * i + j] - (double)cov[6 * j + i]) >
                    1e-6 * (1.0 + std::fabs((double)cov[6 * i + j])))
                    mp_throw(MP_E_ARG, "cov_dT not symmetric");
                A[6 * i + j] = cov[6 * i + j];
            }
        if (!chol6_host(A, L)) mp_throw(MP_E_ARG, "cov_dT not positive semi-definite");
        for (int k = 0; k < 36; ++k) Lf[k] = (float)L[k];
        noise = true;
    }
}

static void run_stage(mp_filter f, int st, int it, hipStream_t s) {
    switch (st) {
        case MP_STAGE_LSH: mp_launch_lsh(f, (uint32_t)f->frame, (uint32_t)it, s); break;
        case MP_STAGE_SORT: mp_launch_sort(f, s); break;
        case MP_STAGE_REFRESH: mp_launch_refresh(f, s); break;
        case MP_STAGE_LIK: mp_launch_likelihood(f, s); break;
        case MP_STAGE_SVGD: mp_launch_svgd(f, s); break;
        case MP_STAGE_POSTERIOR: mp_launch_posterior(f, s); break;
        default: mp_throw(MP_E_ARG, "stage %d cannot run alone", st);
    }
}

// the likelihood and the lists' kernel values at the current (final) poses:
// one likelihood pass and a refresh that only re-ranks the current lists
static void rescore(mp_filter f, hipStream_t s) {
    mp_stage_begin(f, MP_STAGE_LIK);
    run_stage(f, MP_STAGE_LIK, f->p.svgd_iters, s);
    mp_stage_begin(f, MP_STAGE_REFRESH);
    mp_launch_refresh(f, s, 0);
}

void mp_reserve_step(mp_filter f) {
    f->partial.ensure(mp_lik_partial_bytes(f));
    f->red.ensure(std::max(mp_post_scratch_bytes(f), sizeof(uint32_t) * ((size_t)f->n + 64)));
    f->hist.ensure(mp_radix_scratch_bytes(f->n));
}

void mp_step_begin(mp_filter f, bool pred, const float dq[7], const float L[36], bool noise, hipStream_t s) {
    f->clear_flags = true;   // by the step's first kernel
    f->lsh_ahead = false;
    // a captured step always holds the prediction node; it reads whether to
    // predict from the step values
    if (pred || f->dyn) {
        static const float ident[7] = {1, 0, 0, 0, 0, 0, 0};
        static const float zero[36] = {};
        mp_stage_begin(f, MP_STAGE_PREDICT);
        mp_launch_predict(f, pred ? dq : ident, pred ? L : zero, pred && noise, s);
    }
}

// per iteration, in the order of Table II: neighbour list update (LSH, sort,
// refresh; once per hash table, table l of iteration it drawing with counter
// it * tables + l), likelihood evaluation, particle state update
void mp_step_iter_nbr(mp_filter f, int it, hipStream_t s) {
    const int tables = std::max(1, f->p.lsh_tables);
    for (int l = 0; l < tables; ++l)
        for (int st : {MP_STAGE_LSH, MP_STAGE_SORT, MP_STAGE_REFRESH}) {
            mp_stage_begin(f, st);
            if (st == MP_STAGE_LSH && f->lsh_ahead) f->lsh_ahead = false;
            else run_stage(f, st, it * tables + l, s);
        }
}

void mp_step_iter_svgd(mp_filter f, int it, hipStream_t s) {
    mp_stage_begin(f, MP_STAGE_SVGD);
    if (it + 1 < f->p.svgd_iters) {
        const LshArgs next = mp_lsh_args(f, (uint32_t)f->frame, (uint32_t)((it + 1) * std::max(1, f->p.lsh_tables)));
        mp_launch_svgd(f, s, &next);
        f->lsh_ahead = true;
    } else {
        run_stage(f, MP_STAGE_SVGD, it, s);
    }
}

void mp_step_end(mp_filter f, hipStream_t s) {
    const bool corrected = f->scan_n > 0 && f->p.svgd_iters > 0;
    if (corrected) {
        if (f->p.final_rescore) rescore(f, s);
        mp_stage_begin(f, MP_STAGE_POSTERIOR);
    }
    if (mp_take_flags(f)) mp_fill_u32(f->flags.p, 0u, 4, s);   // (neither a prediction nor lists)
    uint64_t* end = nullptr;
    if (f->timing) {
        f->marks.push_back({MP_MARK_END, (int32_t)(kStampMarks + f->marks.size())});
        end = f->stamps.as<uint64_t>() + f->marks.back().slot;
    }
    if (corrected) mp_launch_posterior(f, s, end);
    else if (end && f->marks.size() > 1) mp_launch_stamp(end, s);
}

void mp_step_launches(mp_filter f, bool pred, const float dq[7], const float L[36], bool noise, hipStream_t s) {
    mp_step_begin(f, pred, dq, L, noise, s);
    if (f->scan_n > 0) {
        for (int it = 0; it < f->p.svgd_iters; ++it) {
            mp_step_iter_nbr(f, it, s);
            mp_stage_begin(f, MP_STAGE_LIK);
            run_stage(f, MP_STAGE_LIK, it, s);
            mp_step_iter_svgd(f, it, s);
        }
    }
    mp_step_end(f, s);
}

extern "C" mp_status mp_filter_step(mp_filter f, const float dT[7], const float cov_dT[36], void* stream) {
    return guarded("mp_filter_step", [&]() {
        if (!f) mp_throw(MP_E_ARG, "null filter");
        if (f->scan_n < 0) mp_throw(MP_E_STATE, "mp_filter_step before the first mp_scan_upload");
        if (f->p.scorer == MP_SCORER_SURROGATE && !f->sur)
            mp_throw(MP_E_STATE, "SURROGATE scorer without a network (mp_filter_set_surrogate)");
        hipStream_t s = as_stream(stream);
        float dq[7], L[36];
        bool noise = false;
        if (dT) mp_prepare_prediction(dT, cov_dT, dq, L, noise);
        // every work buffer of the step is sized before anything is launched,
        // so that a failed allocation leaves the filter as it was
        mp_reserve_step(f);
        f->marks.clear();
        // check of the learned scorer (before the step, on the current particles)
        f->sur_fallback = false;
        SurCheck& c = f->chk;
        if (f->p.scorer == MP_SCORER_SURROGATE && c.period > 0 && f->scan_n > 0) {
            if (c.left == 0 && f->frame % c.period == 0) {
                c.last = mp_sur_check(f, c.stride, s);
                ++c.checks;
                if (!(c.last <= c.threshold)) c.left = c.fallback;
            }
            if (c.left > 0) {
                f->sur_fallback = true;
                --c.left;
                ++c.fallback_steps;
            }
        }
        f->timing = true;
        try {
            mp_step_launches(f, dT != nullptr, dq, L, noise, s);
        } catch (...) {
            f->timing = false;
            f->stamp = nullptr;
            f->marks.clear();
            throw;
        }
        f->timing = false;
        f->stamp = nullptr;
        f->step_rec = leave_times(f, f->step_ev, kStampMarks, f->marks.size(), s);
        f->sur_fallback = false;
        f->frame++;
        f->last_stream = s;
    });
}

extern "C" mp_status mp_posterior_query(mp_filter f, mp_posterior* out, float* poses_out, double* weights_out,
                                        void* stream) {
    return guarded("mp_posterior_query", [&]() {
        if (!f || !out) mp_throw(MP_E_ARG, "null argument");
        hipStream_t s = as_stream(stream);
        const size_t N = (size_t)f->n;
        // Poses and weights are packed and checked on the device; outputs on the
        // filter's device are written in place, others go through pinned host
        // memory, query_stage bytes at a time.  (Both copied whole and converted on
        // the host, 1,048,576 particles took 20.3 ms; packed in 36 MiB of device memory
        // and copied from there 2.7 ms, now 2.5, with stages of 0.5 MiB 2.9, of 1 to
        // 16 MiB 2.5 to 2.6; weights alone 0.61 and 0.56, with 1 MiB 0.63.  4096
        // particles 130 us, 28 now, most of it the wait for the stream.)
        std::lock_guard<std::mutex> lock(f->query_mu);
        const auto in_place = [&](const void* p) {
            hipPointerAttribute_t a;
            return p && pointer_attr(p, a) && mp_in_place(a, f->device);
        };
        const bool p_staged = poses_out && !in_place(poses_out), w_staged = weights_out && !in_place(weights_out);
        const bool p_host = p_staged && !is_device_ptr(poses_out), w_host = w_staged && !is_device_ptr(weights_out);
        const size_t per = (p_staged ? sizeof(float) * 7 : 0) + (w_staged ? sizeof(double) : 0);   // bytes of a particle
        const size_t head = 256, room = std::min(per * N, std::max(per, f->query_stage));
        f->host.ensure(head + room);
        char* stage = f->host.as<char>() + head;
        QueryOut* q = f->host.as<QueryOut>();
        static_assert(sizeof(QueryOut) <= 256, "before the packed outputs");
        q->bad = 0;
        const size_t most = per ? room / per : N;   // particles at a time
        for (size_t i0 = 0; i0 < N; i0 += most) {
            const size_t m = std::min(most, N - i0), wbytes = sizeof(double) * m, pbytes = sizeof(float) * 7 * m;
            double* wp = w_staged ? reinterpret_cast<double*>(stage) : (weights_out ? weights_out + i0 : nullptr);
            float* pp = p_staged ? reinterpret_cast<float*>(stage + (w_staged ? wbytes : 0))
                                 : (poses_out ? poses_out + 7 * i0 : nullptr);
            mp_launch_query(f, q, pp, wp, (int32_t)i0, (int32_t)m, s);
            if (p_staged && !p_host) MP_HIP(hipMemcpyAsync(poses_out + 7 * i0, pp, pbytes, hipMemcpyDefault, s));
            if (w_staged && !w_host) MP_HIP(hipMemcpyAsync(weights_out + i0, wp, wbytes, hipMemcpyDefault, s));
            MP_HIP(hipStreamSynchronize(s));
            if (p_host) std::memcpy(poses_out + 7 * i0, pp, pbytes);
            if (w_host) std::memcpy(weights_out + i0, wp, wbytes);
        }
        std::memset(out, 0, sizeof(*out));
        for (int k = 0; k < 7; ++k) out->map_pose[k] = q->pose[k];
        out->map_index = q->index;
        out->map_weight = q->info[4];
        out->n_eff = q->info[5];
        out->log_evidence = q->info[2];
        out->max_loglik = q->info[6];
        out->frame = f->frame;
        out->fp64_resolves = q->resolves;
        out->fallback_steps = f->chk.fallback_steps;
        out->sur_checks = f->chk.checks;
        out->sur_check_ds = f->chk.last;
        const bool finite = all_finite(q->pose, 7) && std::isfinite(q->info[4]) && q->bad == 0;
        if (!finite) mp_throw(MP_E_NUMERIC, "non-finite pose or weight in the filter state");
    });
}

extern "C" mp_status mp_stage_times(mp_filter f, float* ms_out, int32_t* counts_out) {
    return guarded("mp_stage_times", [&]() {
        if (!f || !ms_out) mp_throw(MP_E_ARG, "null argument");
        int32_t counts[MP_NUM_STAGES] = {};
        double ticks[MP_NUM_STAGES] = {};
        if (f->scan_timed || !f->marks.empty()) {
            if ((!f->marks.empty() && !f->step_rec) || (f->scan_timed && !f->scan_rec)) {   // not asked for before
                f->times.ensure(f->stamps.bytes);
                if (!f->step_ev) MP_HIP(hipEventCreateWithFlags(&f->step_ev, hipEventDisableTiming));
                if (!f->scan_ev) MP_HIP(hipEventCreateWithFlags(&f->scan_ev, hipEventDisableTiming));
                MP_HIP(hipDeviceSynchronize());
                MP_HIP(hipMemcpy(f->times.p, f->stamps.p, f->stamps.bytes, hipMemcpyDeviceToHost));
                f->step_rec = f->scan_rec = true;   // (an event that was never recorded is over)
            } else {
                if (!f->marks.empty()) MP_HIP(hipEventSynchronize(f->step_ev));
                if (f->scan_timed) MP_HIP(hipEventSynchronize(f->scan_ev));
            }
            const uint64_t* t = f->times.as<uint64_t>();
            auto add = [&](int st, uint64_t from, uint64_t to, bool count) {
                ticks[st] += to > from ? (double)(to - from) : 0.0;
                counts[st] += count ? 1 : 0;
            };
            if (f->scan_timed) add(MP_STAGE_SCAN, t[0], t[1], true);
            for (size_t k = 0; k + 1 < f->marks.size(); ++k) {
                const uint64_t from = t[f->marks[k].slot], to = t[f->marks[k + 1].slot];
                const int st = f->marks[k].stage;
                // the likelihood: walk order, then its kernel, then the solve
                if (st == MP_STAGE_LIK_CORE || st == MP_MARK_SOLVE) add(MP_STAGE_LIK, from, to, false);
                if (st != MP_MARK_SOLVE) add(st, from, to, true);
            }
        }
        int dev = 0, khz = 0;
        MP_HIP(hipGetDevice(&dev));
        MP_HIP(hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev));
        for (int st = 0; st < MP_NUM_STAGES; ++st) {
            ms_out[st] = (float)(ticks[st] / (double)std::max(1, khz));
            if (counts_out) counts_out[st] = counts[st];
        }
    });
}

// ------------------------------------------------------------ debug access
struct NamedBuf {
    void* p;
    size_t bytes;
    bool settable;
};

static NamedBuf lookup_buf(mp_filter f, const char* name) {
    const size_t N = (size_t)f->n, K = (size_t)f->K;
    const std::string s(name ? name : "");
    if (s == "poses") return {f->poses[f->cur].p, 32 * N, true};
    if (s == "psi") return {f->psi.p, 32 * N, true};
    if (s == "hb") {
        f->hb.ensure(28 * 4 * N);
        return {f->hb.p, 28 * 4 * N, false};
    }
    if (s == "solve") {
        f->solve_how.ensure(4 * N);
        return {f->solve_how.p, 4 * N, false};
    }
    if (s == "codes") return {f->codes.p, 4 * N, true};
    if (s == "sorted") return {f->sorted.p, 4 * N, true};
    if (s == "scodes") return {f->scodes.p, 4 * N, true};
    if (s == "head") return {f->head.p, 4 * N, true};
    if (s == "end") return {f->end.p, 4 * N, true};
    if (s == "nbr") return {f->nbr.p, 4 * K * N, true};
    if (s == "kval") return {f->kval.p, 4 * K * N, true};
    if (s == "cnt") return {f->cnt.p, 4 * N, true};
    if (s == "prior") return {f->prior.p, 4 * N, true};
    if (s == "post") return {f->prior.p, 4 * N, false};
    if (s == "post0") return {f->post0.p, 4 * N, false};
    if (s == "scan") return {f->scan_orig.p, f->scan_n > 0 ? 48 * (size_t)f->scan_n : 0, false};
    if (s == "scan_walk") return {f->scan.p, f->scan_n > 0 ? 48 * (size_t)f->scan_n : 0, false};
    if (s == "odo_nn") return {f->odo_nn.p, f->odo_nn.p && f->scan_n > 0 ? 4 * (size_t)f->scan_n : 0, false};
    if (s == "tlsh") return {f->tlsh.p, 32, false};
    if (s == "sort_wait") return {f->hist.p ? (void*)mp_radix_wait_flag(f->hist) : nullptr, f->hist.p ? 4u : 0u, false};
    mp_throw(MP_E_ARG, "unknown buffer '%s'", s.c_str());
}

extern "C" mp_status mp_debug_get(mp_filter f, const char* name, void* dst, int64_t bytes, void* stream) {
    return guarded("mp_debug_get", [&]() {
        if (!f || !dst) mp_throw(MP_E_ARG, "null argument");
        const NamedBuf b = lookup_buf(f, name);
        if ((size_t)bytes != b.bytes) mp_throw(MP_E_ARG, "'%s' holds %zu bytes, asked %lld", name, b.bytes, (long long)bytes);
        hipStream_t s = as_stream(stream);
        copy_out(dst, b.p, b.bytes, s);
        MP_HIP(hipStreamSynchronize(s));
    });
}

extern "C" mp_status mp_debug_set(mp_filter f, const char* name, const void* src, int64_t bytes, void* stream) {
    return guarded("mp_debug_set", [&]() {
        if (!f || !src) mp_throw(MP_E_ARG, "null argument");
        hipStream_t s = as_stream(stream);
        if (std::string(name ? name : "") == "capture_hb") {
            if (bytes != 4) mp_throw(MP_E_ARG, "capture_hb takes one int32");
            int32_t v = 0;
            fetch_host(src, 4, &v, s);
            f->capture_hb = v ? 1 : 0;
            if (f->capture_hb) f->hb.ensure(28 * 4 * (size_t)f->n);
            if (f->capture_hb) f->solve_how.ensure(4 * (size_t)f->n);
            return;
        }
        if (std::string(name ? name : "") == "query_stage") {
            if (bytes != 4) mp_throw(MP_E_ARG, "query_stage takes one int32");
            int32_t v = 0;
            fetch_host(src, 4, &v, s);
            if (v < 0) mp_throw(MP_E_ARG, "query_stage must not be negative");
            f->query_stage = (size_t)v;
            return;
        }
        const NamedBuf b = lookup_buf(f, name);
        if (!b.settable) mp_throw(MP_E_ARG, "'%s' is read-only", name);
        if ((size_t)bytes != b.bytes) mp_throw(MP_E_ARG, "'%s' holds %zu bytes, given %lld", name, b.bytes, (long long)bytes);
        MP_HIP(hipMemcpyAsync(b.p, src, b.bytes, hipMemcpyDefault, s));
        MP_HIP(hipStreamSynchronize(s));
        if (b.p == f->sorted.p) f->rank_set = false;
    });
}

extern "C" mp_status mp_debug_stage(mp_filter f, int32_t stage, int32_t iteration, const float dT[7],
                                    const float cov_dT[36], void* stream) {
    return guarded("mp_debug_stage", [&]() {
        if (!f) mp_throw(MP_E_ARG, "null filter");
        hipStream_t s = as_stream(stream);
        if (stage == MP_STAGE_PREDICT) {
            if (!dT) mp_throw(MP_E_ARG, "prediction needs dT");
            float dq[7], L[36];
            bool noise = false;
            mp_prepare_prediction(dT, cov_dT, dq, L, noise);
            mp_launch_predict(f, dq, L, noise, s);
        } else if (stage == MP_DEBUG_RESCORE) {
            if (f->scan_n < 0) mp_throw(MP_E_STATE, "no scan uploaded");
            MP_HIP(hipMemsetAsync(f->flags.p, 0, 16, s));
            rescore(f, s);
        } else {
            if ((stage == MP_STAGE_LIK) && f->scan_n < 0) mp_throw(MP_E_STATE, "no scan uploaded");
            if (stage == MP_STAGE_LIK) MP_HIP(hipMemsetAsync(f->flags.p, 0, 16, s));
            run_stage(f, stage, iteration, s);
        }
        MP_HIP(hipStreamSynchronize(s));
    });
}

// ------------------------------------------------------------ surrogate
extern "C" void mp_surrogate_default_params(mp_surrogate_params* p) {
    if (!p) return;
    std::memset(p, 0, sizeof(*p));
    p->f_max = 0.0f;
    p->sigma_s = 0.03f;
    p->d_max = 0.0f;
    p->c_max = 9.0f;
    p->lr = 1e-3f;
    p->lr_min = 1e-5f;
    p->beta1 = 0.9f;
    p->beta2 = 0.999f;
    p->adam_eps = 1e-8f;
    p->total_steps = 20000;
    p->batch = 65536;
    p->seed = 1;
}

extern "C" mp_status mp_surrogate_create(mp_map map, const mp_surrogate_params* params, void* stream,
                                         mp_surrogate* out) {
    return guarded("mp_surrogate_create", [&]() {
        if (!map || !params || !out) mp_throw(MP_E_ARG, "null argument");
        mp_surrogate_params p = *params;
        const float fs[] = {p.box_min[0], p.box_min[1], p.box_min[2], p.box_max[0], p.box_max[1], p.box_max[2],
                            p.f_max, p.sigma_s, p.d_max, p.c_max, p.lr, p.lr_min, p.beta1, p.beta2, p.adam_eps};
        for (float v : fs)
            if (!std::isfinite(v)) mp_throw(MP_E_ARG, "non-finite parameter");
        if (!(p.sigma_s > 0) || p.d_max < 0 || !(p.c_max > 0) || p.f_max < 0 || !(p.lr > 0) || p.lr_min < 0 ||
            !(p.beta1 >= 0 && p.beta1 < 1) || !(p.beta2 >= 0 && p.beta2 < 1) || !(p.adam_eps > 0) ||
            p.total_steps < 1 || p.batch < 256 || p.batch > (1 << 20))
            mp_throw(MP_E_ARG, "parameter out of range");
        const float r = map->params.voxel;
        if (p.d_max == 0.0f) p.d_max = 2.0f * r;
        bool box_given = false;
        for (int a = 0; a < 3; ++a) box_given = box_given || p.box_min[a] != p.box_max[a];
        if (!box_given) {
            if (map->info.num_gauss <= 0) mp_throw(MP_E_ARG, "empty map and no feature box");
            for (int a = 0; a < 3; ++a) {
                p.box_min[a] = map->info.box_min[a];
                p.box_max[a] = map->info.box_max[a];
            }
        }
        double ext = 0.0;
        for (int a = 0; a < 3; ++a) {
            if (!(p.box_max[a] > p.box_min[a])) mp_throw(MP_E_ARG, "empty feature box");
            ext = std::max(ext, (double)p.box_max[a] - (double)p.box_min[a]);
        }
        if (p.f_max == 0.0f) p.f_max = (float)(ext / (double)r);
        if (!(p.f_max >= 1.0f)) mp_throw(MP_E_ARG, "f_max below one cycle per box");
        auto S = std::make_unique<mp_surrogate_s>();
        S->map = map;
        S->p = p;
        mp_surrogate_info& I = S->info;
        std::memset(&I, 0, sizeof(I));
        I.n_params = MP_SUR_NPARAMS;
        for (int a = 0; a < 3; ++a) {
            I.lo[a] = p.box_min[a];
            I.inv_ext[a] = (float)(1.0 / ext);
        }
        for (int l = 0; l < 32; ++l) I.freqs[l] = (float)std::pow((double)p.f_max, (double)l / 31.0);
        const double eps = map->params.cov_eps, s2 = (double)p.sigma_s * (double)p.sigma_s;
        I.r_scale = mp_residual_r_out(p.d_max, p.sigma_s, map->params.cov_eps);
        I.g_scale = (float)(1.0 / std::sqrt(eps + s2));
        I.weight_bytes = MP_SUR_IMAGE_BYTES;
        hipStream_t s = as_stream(stream);
        mp_sur_alloc(S.get(), s);
        mp_sur_init_weights(S.get(), s);
        MP_HIP(hipStreamSynchronize(s));
        map->users++;
        *out = S.release();
    });
}

extern "C" mp_status mp_surrogate_destroy(mp_surrogate sur) {
    return guarded("mp_surrogate_destroy", [&]() {
        if (!sur) return;
        if (sur->users > 0) mp_throw(MP_E_STATE, "network still used by %d filter(s)", sur->users);
        MP_HIP(hipDeviceSynchronize());
        if (sur->map) sur->map->users--;
        delete sur;
    });
}

extern "C" mp_status mp_surrogate_get_info(mp_surrogate sur, mp_surrogate_info* out) {
    return guarded("mp_surrogate_get_info", [&]() {
        if (!sur || !out) mp_throw(MP_E_ARG, "null argument");
        *out = sur->info;
    });
}

static void check_points(const float* xyz, int64_t n) {
    if (n < 0 || (n > 0 && !xyz)) mp_throw(MP_E_ARG, "bad point array");
    if (n > ((int64_t)1 << 31)) mp_throw(MP_E_ARG, "too many points");
}

extern "C" mp_status mp_surrogate_label(mp_surrogate sur, const float* xyz, int64_t n, float* out4, void* stream) {
    return guarded("mp_surrogate_label", [&]() {
        if (!sur) mp_throw(MP_E_ARG, "null surrogate");
        check_points(xyz, n);
        if (n > 0 && !out4) mp_throw(MP_E_ARG, "null output");
        if (n == 0) return;
        hipStream_t s = as_stream(stream);
        DevMem tin, tout;
        const float* d = static_cast<const float*>(stage_in(xyz, sizeof(float) * 3 * (size_t)n, tin, s));
        const bool dev_out = is_device_ptr(out4);
        float* o = out4;
        if (!dev_out) {
            tout.alloc(sizeof(float) * 4 * (size_t)n);
            o = tout.as<float>();
        }
        mp_sur_label(sur, d, n, o, false, s);
        if (!dev_out) copy_out(out4, o, sizeof(float) * 4 * (size_t)n, s);
        MP_HIP(hipStreamSynchronize(s));
    });
}

extern "C" mp_status mp_surrogate_eval(mp_surrogate sur, const float* xyz, int64_t n, float* out4, void* stream) {
    return guarded("mp_surrogate_eval", [&]() {
        if (!sur) mp_throw(MP_E_ARG, "null surrogate");
        check_points(xyz, n);
        if (n > 0 && !out4) mp_throw(MP_E_ARG, "null output");
        if (n == 0) return;
        hipStream_t s = as_stream(stream);
        DevMem tin, tout;
        const float* d = static_cast<const float*>(stage_in(xyz, sizeof(float) * 3 * (size_t)n, tin, s));
        const bool dev_out = is_device_ptr(out4);
        float* o = out4;
        if (!dev_out) {
            tout.alloc(sizeof(float) * 4 * (size_t)n);
            o = tout.as<float>();
        }
        mp_sur_eval(sur, d, n, o, s);
        if (!dev_out) copy_out(out4, o, sizeof(float) * 4 * (size_t)n, s);
        MP_HIP(hipStreamSynchronize(s));
    });
}

extern "C" mp_status mp_surrogate_set_data(mp_surrogate sur, const float* xyz, int64_t n, void* stream) {
    return guarded("mp_surrogate_set_data", [&]() {
        if (!sur) mp_throw(MP_E_ARG, "null surrogate");
        check_points(xyz, n);
        if (n < 1) mp_throw(MP_E_ARG, "training set must hold at least one point");
        hipStream_t s = as_stream(stream);
        sur->dxyz.alloc(sizeof(float) * 3 * (size_t)n);
        sur->dlab.alloc(sizeof(float) * 4 * (size_t)n);
        MP_HIP(hipMemcpyAsync(sur->dxyz.p, xyz, sizeof(float) * 3 * (size_t)n, hipMemcpyDefault, s));
        mp_sur_label(sur, sur->dxyz.as<float>(), n, sur->dlab.as<float>(), true, s);
        sur->info.n_data = n;
        MP_HIP(hipStreamSynchronize(s));
    });
}

extern "C" mp_status mp_surrogate_train(mp_surrogate sur, int32_t steps, float* loss_out, void* stream) {
    return guarded("mp_surrogate_train", [&]() {
        if (!sur) mp_throw(MP_E_ARG, "null surrogate");
        if (steps < 0) mp_throw(MP_E_ARG, "negative step count");
        if (sur->info.n_data < 1) mp_throw(MP_E_STATE, "no training data (mp_surrogate_set_data)");
        if (steps == 0) return;
        hipStream_t s = as_stream(stream);
        const bool full = sur->info.n_data <= sur->p.batch;
        const int32_t n_real = full ? (int32_t)sur->info.n_data : sur->p.batch;
        mp_sur_ensure_batch(sur, n_real);
        sur->losses.ensure(sizeof(float) * (size_t)steps);
        const mp_surrogate_params& p = sur->p;
        for (int32_t k = 0; k < steps; ++k) {
            const int64_t t = sur->info.steps;   // steps taken before this one
            const double frac = std::min(1.0, (double)t / (double)p.total_steps);
            const double lr = p.lr_min + 0.5 * ((double)p.lr - p.lr_min) * (1.0 + std::cos(M_PI * frac));
            mp_sur_train_step(sur, n_real, full, (uint32_t)t, (float)lr, sur->losses.as<float>() + k, s);
        }
        if (loss_out) {
            MP_HIP(hipMemcpyAsync(loss_out, sur->losses.p, sizeof(float) * (size_t)steps, hipMemcpyDeviceToHost, s));
            MP_HIP(hipStreamSynchronize(s));
        }
    });
}

extern "C" mp_status mp_surrogate_grad(mp_surrogate sur, const float* xyz, const float* target4, int64_t n,
                                       float* grad_out, float* loss_out, void* stream) {
    return guarded("mp_surrogate_grad", [&]() {
        if (!sur || !xyz || !target4) mp_throw(MP_E_ARG, "null argument");
        if (n < 1 || n > sur->p.batch) mp_throw(MP_E_ARG, "n must be 1..batch");
        hipStream_t s = as_stream(stream);
        mp_sur_ensure_batch(sur, n);
        std::vector<float> tgt(4 * (size_t)n);
        fetch_host(target4, sizeof(float) * 4 * (size_t)n, tgt.data(), s);
        const float is = 1.0f / sur->info.r_scale, ig = 1.0f / sur->info.g_scale;
        for (int64_t i = 0; i < n; ++i) {
            tgt[4 * i] *= is;
            for (int a = 1; a < 4; ++a) tgt[4 * i + a] *= ig;
        }
        const int32_t bp = sur->cap;
        MP_HIP(hipMemsetAsync(sur->bxyz.p, 0, sizeof(float) * 3 * (size_t)bp, s));
        MP_HIP(hipMemsetAsync(sur->btgt.p, 0, sizeof(float) * 4 * (size_t)bp, s));
        MP_HIP(hipMemcpyAsync(sur->bxyz.p, xyz, sizeof(float) * 3 * (size_t)n, hipMemcpyDefault, s));
        MP_HIP(hipMemcpyAsync(sur->btgt.p, tgt.data(), sizeof(float) * 4 * (size_t)n, hipMemcpyHostToDevice, s));
        sur->losses.ensure(sizeof(float));
        mp_sur_grad_step(sur, (int32_t)n, false, 0.0f, sur->losses.as<float>(), s);
        if (grad_out) copy_out(grad_out, sur->G.p, sizeof(float) * MP_SUR_NPARAMS, s);
        if (loss_out) MP_HIP(hipMemcpyAsync(loss_out, sur->losses.p, sizeof(float), hipMemcpyDeviceToHost, s));
        MP_HIP(hipStreamSynchronize(s));
    });
}

extern "C" mp_status mp_surrogate_get_params(mp_surrogate sur, float* params, void* stream) {
    return guarded("mp_surrogate_get_params", [&]() {
        if (!sur || !params) mp_throw(MP_E_ARG, "null argument");
        hipStream_t s = as_stream(stream);
        copy_out(params, sur->P.p, sizeof(float) * MP_SUR_NPARAMS, s);
        MP_HIP(hipStreamSynchronize(s));
    });
}

extern "C" mp_status mp_surrogate_set_params(mp_surrogate sur, const float* params, void* stream) {
    return guarded("mp_surrogate_set_params", [&]() {
        if (!sur || !params) mp_throw(MP_E_ARG, "null argument");
        hipStream_t s = as_stream(stream);
        std::vector<float> h(MP_SUR_NPARAMS);
        fetch_host(params, sizeof(float) * MP_SUR_NPARAMS, h.data(), s);
        if (!all_finite(h.data(), h.size())) mp_throw(MP_E_ARG, "non-finite weights");
        MP_HIP(hipMemcpyAsync(sur->P.p, h.data(), sizeof(float) * MP_SUR_NPARAMS, hipMemcpyHostToDevice, s));
        mp_sur_reset_adam(sur, s);
        mp_sur_publish(sur, s);
        MP_HIP(hipStreamSynchronize(s));
    });
}

extern "C" mp_status mp_filter_set_surrogate_check(mp_filter f, int32_t period, int32_t stride, float threshold,
                                                   int32_t fallback) {
    return guarded("mp_filter_set_surrogate_check", [&]() {
        if (!f) mp_throw(MP_E_ARG, "null filter");
        if (period < 0 || stride < 1 || fallback < 0 || !(threshold >= 0.0f) || !std::isfinite(threshold))
            mp_throw(MP_E_ARG, "period >= 0, stride >= 1, fallback >= 0 and a finite threshold >= 0 expected");
        if (f->batch_users > 0) mp_throw(MP_E_STATE, "filter held by a batch");
        SurCheck& c = f->chk;
        c.period = period;
        c.stride = stride;
        c.threshold = threshold;
        c.fallback = fallback;
        c.left = 0;
    });
}

extern "C" mp_status mp_filter_set_surrogate(mp_filter f, mp_surrogate sur) {
    return guarded("mp_filter_set_surrogate", [&]() {
        if (!f) mp_throw(MP_E_ARG, "null filter");
        if (sur && sur->map != f->map) mp_throw(MP_E_ARG, "network built for another map");
        if (f->sur) f->sur->users--;
        f->sur = sur;
        if (sur) sur->users++;
    });
}
