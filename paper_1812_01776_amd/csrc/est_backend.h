// Device-side services the host planner needs: memory, copies, kernel launches, events.
// Implemented for the GPU in est_kernels.hip.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include "est_types.h"

namespace estbe {

int init();                       // 0, or non-zero with last_error() set when no usable GPU is present
const char *last_error();
void *dmalloc(size_t bytes);      // nullptr on failure
void dfree(void *p);
size_t mem_free();                // free device memory in bytes
int h2d(void *dst, const void *src, size_t bytes, void *stream);
int d2h(void *dst, const void *src, size_t bytes, void *stream);
int d2d(void *dst, const void *src, size_t bytes, void *stream);
int zero(void *dst, size_t bytes, void *stream);
int sync(void *stream);

int launch_cfg(const EstCfgArgs &a, void *stream);
int launch_prep1(const EstPrepArgs &a, void *stream);
int launch_prep2(const EstPrepArgs &a, void *stream);
int launch_sim(const EstSimArgs &a, void *stream);
// The envelope's launch, one wavefront per a.per_wave queries and width, four to a workgroup: as many consecutive queries per
// wavefront as keep twice the wavefronts the device holds (16,384), at most eight blocks of 64, and beyond that as many as keep the
// launch at 2^25 wavefronts: it would have 2^32 work-items, one more than a launch can have, from queries x widths = 2^35 on.
inline uint32_t envelope_per_wave(uint64_t n, uint32_t n_win) {
    const uint64_t blocks = (n + 63) / 64;
    uint64_t k = n / 64 * n_win / 16384;
    k = k < 1 ? 1 : k > 8 ? 8 : k;
    const uint64_t most = (1u << 25) / n_win;  // wavefronts of one width
    if ((blocks + k - 1) / k > most) k = (blocks + most - 1) / most;
    return (uint32_t)(64 * k);
}
inline uint32_t envelope_groups(uint64_t n, uint32_t n_win, uint32_t per_wave) {
    return (uint32_t)(((n + per_wave - 1) / per_wave * n_win + 3) / 4);
}
int launch_envelope(const EstEnvArgs &a, void *stream);
// workgroups of the simulation kernel the device holds at once: waves wavefronts and lds_bytes of LDS each, the build for
// waves_per_simd (4 or 6) wavefronts per SIMD; 0 when it does not fit
uint32_t max_resident_groups(uint32_t waves, uint32_t lds_bytes, uint32_t waves_per_simd);

void *stream_create();            // a second stream at the default priority; nullptr on failure
void stream_destroy(void *stream);
int stream_wait_event(void *stream, void *ev);  // later work on stream starts after ev has completed

// The library's own fixed scratch on the current device (a file-scope device array, resolved once per
// device): its address and size, or nullptr with last_error() set.  Nothing is allocated.
void *static_scratch(uint64_t *bytes);
void *host_pinned_alloc(size_t bytes);  // page-locked host memory; nullptr on failure
void host_pinned_free(void *p);

void *event_create();
void event_destroy(void *ev);
int event_record(void *ev, void *stream);
float event_ms(void *start, void *stop);  // both must have completed

}  // namespace estbe
