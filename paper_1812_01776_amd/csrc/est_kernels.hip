// GPU back end: kernel entry points and the HIP runtime
// calls the host planner needs.  gfx950 only.
#include <hip/hip_runtime.h>

#include <stdlib.h>

#include <string>

#include "est_backend.h"
#include "wave_gfx950.h"
#include "est_device.h"

namespace {

thread_local std::string g_err;

int check(hipError_t e, const char *what) {
    if (e == hipSuccess) return 0;
    g_err = std::string(what) + ": " + hipGetErrorString(e);
    return 1;
}

// The simulation kernel (see the driver in est_device.h).  The register budget is pinned per build: WAVES_PER_SIMD
// resident wavefronts per SIMD, 128 or 80 registers per lane.  Every wait is bounded: a wavefront of a workgroup in which nothing
// moves any more, or that sees that another one gave up, sets the error flag and leaves.
constexpr uint32_t STILL_LIMIT = 1u << 18;  // looks of about four microseconds each
template <bool DIAG, int WAVES_PER_SIMD, bool MEMO>
__global__ __launch_bounds__(64 * EST_MAX_WAVES) __attribute__((amdgpu_waves_per_eu(WAVES_PER_SIMD, WAVES_PER_SIMD)))
void est_sim_kernel(EstSimArgs a) {
    extern __shared__ uint64_t lds[];  // a.shared_bytes, then a.lds_bytes per wavefront
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint64_t *my_lds = lds + a.shared_bytes / 8 + (size_t)wave * (a.lds_bytes / 8);
    const estdev::Pool p = estdev::make_pool(a, (uint32_t *)lds);
    if (wave == 0) estdev::pool_setup(p);
    __syncthreads();
    uint32_t at = 0;
    for (estdev::Wait wait = {0, 0, 0};;) {
        const uint32_t r = estdev::pool_step<DIAG, MEMO>(p, blockIdx.x, wave, at, my_lds);
        if (r == estdev::STEP_END) break;
        if (r == estdev::STEP_WORKED) {
            wait.idle = 0;
            continue;
        }
        ++wait.idle;
        if (estdev::stuck(p, wait, STILL_LIMIT) || ((wait.idle & 255u) == 0u && wv::load_shared(&a.status->sim_error))) {
            if (wv::lane() == 0) a.status->sim_error = 1;
            break;
        }
        // (look again soon at first, then leave the issue slots to those that work)
        if (wait.idle < 8u) __builtin_amdgcn_s_sleep(8);
        else if (wait.idle < 32u) __builtin_amdgcn_s_sleep(32);
        else __builtin_amdgcn_s_sleep(127);
    }
}

__global__ __launch_bounds__(256) void est_prep1_kernel(EstPrepArgs a) {
    estdev::prep1_thread(a, blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
}

__global__ __launch_bounds__(256) void est_prep2_kernel(EstPrepArgs a) {
    estdev::prep2_thread(a, blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
}

__global__ __launch_bounds__(256) void est_envelope_kernel(EstEnvArgs a) {
    const uint32_t w = __builtin_amdgcn_readfirstlane(blockIdx.x * 4u + (threadIdx.x >> 6));
    const uint64_t j0 = (uint64_t)(w / a.n_win) * a.per_wave;  // (the widths of the same queries side by side: they read the same arrivals)
    if (j0 < a.n) estdev::envelope_wave(a, w % a.n_win, (uint32_t)j0, (uint32_t)(j0 + a.per_wave < a.n ? j0 + a.per_wave : a.n));
}

__global__ __launch_bounds__(256) void est_cfg_kernel(EstCfgArgs a) {
    estdev::cfg_thread(a, blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
}

// Scratch of estimator_run_static_dev, the entry point for callers that cannot allocate: every GPU the
// library runs on holds this array until the process ends.  In host code the array's name is only a
// symbol: its device address is asked for once per device (static_scratch below) and used from then on.
static __device__ __align__(256) unsigned char scratch[EST_STATIC_SCRATCH_BYTES];
constexpr int MAX_DEVICES = 64;
void *g_scratch_ptr[MAX_DEVICES];

uint32_t blocks_for(uint64_t items, uint32_t per_block, uint32_t max_blocks) {
    uint64_t b = (items + per_block - 1) / per_block;
    if (b < 1) b = 1;
    return (uint32_t)(b > max_blocks ? max_blocks : b);
}

}  // namespace

namespace estbe {

const char *last_error() { return g_err.c_str(); }

int init() {
    int n = 0;
    if (check(hipGetDeviceCount(&n), "hipGetDeviceCount")) return 1;
    if (n < 1) {
        g_err = "no HIP device";
        return 1;
    }
    return 0;
}

void *dmalloc(size_t bytes) {
    void *p = nullptr;
    if (check(hipMalloc(&p, bytes), "hipMalloc")) {
        (void)hipGetLastError();  // (the caller may try again smaller: no stale error for the next launch check to find)
        return nullptr;
    }
    return p;
}

void dfree(void *p) { (void)hipFree(p); }

size_t mem_free() {
    size_t f = 0, t = 0;
    if (hipMemGetInfo(&f, &t) != hipSuccess) return 0;
    return f;
}

int h2d(void *dst, const void *src, size_t bytes, void *stream) {
    if (bytes == 0) return 0;
    return check(hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, (hipStream_t)stream), "hipMemcpyAsync H2D");
}
int d2h(void *dst, const void *src, size_t bytes, void *stream) {
    if (bytes == 0) return 0;
    return check(hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, (hipStream_t)stream), "hipMemcpyAsync D2H");
}
int d2d(void *dst, const void *src, size_t bytes, void *stream) {
    if (bytes == 0) return 0;
    return check(hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToDevice, (hipStream_t)stream), "hipMemcpyAsync D2D");
}
int zero(void *dst, size_t bytes, void *stream) {
    if (bytes == 0) return 0;
    return check(hipMemsetAsync(dst, 0, bytes, (hipStream_t)stream), "hipMemsetAsync");
}
int sync(void *stream) { return check(hipStreamSynchronize((hipStream_t)stream), "hipStreamSynchronize"); }

int launch_cfg(const EstCfgArgs &a, void *stream) {
    est_cfg_kernel<<<blocks_for(a.n_cfg, 256, 1024), 256, 0, (hipStream_t)stream>>>(a);
    return check(hipGetLastError(), "est_cfg_kernel");
}
int launch_prep1(const EstPrepArgs &a, void *stream) {
    est_prep1_kernel<<<blocks_for(a.n, 256 * 8, 1024), 256, 0, (hipStream_t)stream>>>(a);
    return check(hipGetLastError(), "est_prep1_kernel");
}
int launch_prep2(const EstPrepArgs &a, void *stream) {
    est_prep2_kernel<<<blocks_for(a.n, 256, 4096), 256, 0, (hipStream_t)stream>>>(a);
    return check(hipGetLastError(), "est_prep2_kernel");
}
int launch_envelope(const EstEnvArgs &a, void *stream) {
    est_envelope_kernel<<<envelope_groups(a.n, a.n_win, a.per_wave), 256, 0, (hipStream_t)stream>>>(a);
    return check(hipGetLastError(), "est_envelope_kernel");
}
int launch_sim(const EstSimArgs &a, void *stream) {
    const uint32_t groups = (a.n_slots + a.per_group - 1) / a.per_group;
    const size_t lds = (size_t)a.shared_bytes + (size_t)a.lds_bytes * a.waves;
    const dim3 grid(groups), block(64 * a.waves);
    if (a.waves < 1 || a.waves > EST_MAX_WAVES || a.per_group < 1 || a.per_group > a.waves || groups < 1) {
        g_err = "est_sim_kernel: launch shape";
        return 1;
    }
    // (the variant that keeps diagnostic counters is launched only when they are asked for, the one for candidates that skip
    // operations when some do)
    if (a.skip_ops) {
        if (a.waves_per_simd == 6)
            est_sim_kernel<false, 6, true><<<grid, block, lds, (hipStream_t)stream>>>(a);
        else
            est_sim_kernel<false, 4, true><<<grid, block, lds, (hipStream_t)stream>>>(a);
    } else if (a.dbg_ticks)
        est_sim_kernel<true, 4, false><<<grid, block, lds, (hipStream_t)stream>>>(a);
    else if (a.waves_per_simd == 6)
        est_sim_kernel<false, 6, false><<<grid, block, lds, (hipStream_t)stream>>>(a);
    else
        est_sim_kernel<false, 4, false><<<grid, block, lds, (hipStream_t)stream>>>(a);
    return check(hipGetLastError(), "est_sim_kernel");
}

uint32_t max_resident_groups(uint32_t waves, uint32_t lds_bytes, uint32_t waves_per_simd) {
    int dev = 0, cus = 0, blocks = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    const hipError_t e = waves_per_simd == 6
                             ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, est_sim_kernel<false, 6, false>, 64 * (int)waves, lds_bytes)
                             : hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, est_sim_kernel<false, 4, false>, 64 * (int)waves, lds_bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return (uint32_t)cus * (uint32_t)(blocks > 0 ? blocks : 0);
}

void *stream_create() {
    hipStream_t st = nullptr;
    if (check(hipStreamCreateWithFlags(&st, hipStreamNonBlocking), "hipStreamCreate")) return nullptr;
    return (void *)st;
}
void stream_destroy(void *stream) { (void)hipStreamDestroy((hipStream_t)stream); }
int stream_wait_event(void *stream, void *ev) { return check(hipStreamWaitEvent((hipStream_t)stream, (hipEvent_t)ev, 0), "hipStreamWaitEvent"); }

void *static_scratch(uint64_t *bytes) {
    int dev = 0;
    if (check(hipGetDevice(&dev), "hipGetDevice")) return nullptr;
    if (dev < 0 || dev >= MAX_DEVICES) {
        g_err = "device index out of range for the static scratch";
        return nullptr;
    }
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (check(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)), "hipGetSymbolAddress(scratch)")) return nullptr;
        g_scratch_ptr[dev] = p;
    }
    if (bytes) *bytes = EST_STATIC_SCRATCH_BYTES;
    return g_scratch_ptr[dev];
}

void *host_pinned_alloc(size_t bytes) {
    void *p = nullptr;
    if (check(hipHostMalloc(&p, bytes, hipHostMallocDefault), "hipHostMalloc")) return nullptr;
    return p;
}
void host_pinned_free(void *p) { (void)hipHostFree(p); }

void *event_create() {
    hipEvent_t e = nullptr;
    if (check(hipEventCreate(&e), "hipEventCreate")) return nullptr;
    return (void *)e;
}
void event_destroy(void *ev) { (void)hipEventDestroy((hipEvent_t)ev); }
int event_record(void *ev, void *stream) { return check(hipEventRecord((hipEvent_t)ev, (hipStream_t)stream), "hipEventRecord"); }
float event_ms(void *start, void *stop) {
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, (hipEvent_t)start, (hipEvent_t)stop) != hipSuccess) return 0.f;
    return ms;
}

}  // namespace estbe
