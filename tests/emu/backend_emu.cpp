// Host back end for the lock-step wavefront emulation (test infrastructure): "device" memory is
// host memory, a kernel launch runs every wavefront as 64 fibers, one wavefront after the other.
#include <string.h>
#include <ucontext.h>

#include <functional>
#include <string>
#include <vector>

#include "wave_emu.h"
#include "../../paper_1812_01776_amd/csrc/est_backend.h"
#include "../../paper_1812_01776_amd/csrc/est_device.h"

namespace emu {

namespace {
const size_t STACK = 256 * 1024;
ucontext_t g_sched, g_ctx[64];
std::vector<char> g_stacks;
bool g_done[64];
uint32_t g_cur;
uint64_t g_x[2][64];
uint32_t g_tag[64];
uint32_t g_nb[64];
const std::function<void()> *g_body;

void trampoline() {
    (*g_body)();
    g_done[g_cur] = true;
    swapcontext(&g_ctx[g_cur], &g_sched);
}
}  // namespace

uint32_t lane() { return g_cur; }

const uint64_t *exchange(uint64_t v, uint32_t tag) {
    const uint32_t me = g_cur;
    const uint32_t ph = g_nb[me] & 1u;
    g_x[ph][me] = v;
    g_tag[me] = tag;
    g_nb[me]++;
    swapcontext(&g_ctx[me], &g_sched);  // wait for the other lanes
    g_cur = me;
    return g_x[ph];
}

void run_wave(const std::function<void()> &body) {
    if (g_stacks.empty()) g_stacks.resize(64 * STACK);
    g_body = &body;
    for (int l = 0; l < 64; ++l) {
        g_done[l] = false;
        g_nb[l] = 0;
        getcontext(&g_ctx[l]);
        g_ctx[l].uc_stack.ss_sp = g_stacks.data() + (size_t)l * STACK;
        g_ctx[l].uc_stack.ss_size = STACK;
        g_ctx[l].uc_link = &g_sched;
        makecontext(&g_ctx[l], trampoline, 0);
    }
    for (;;) {
        int ndone = 0;
        for (int l = 0; l < 64; ++l) {
            if (g_done[l]) { ++ndone; continue; }
            g_cur = (uint32_t)l;
            swapcontext(&g_sched, &g_ctx[l]);
            if (g_done[l]) ++ndone;
        }
        if (ndone == 64) break;
        if (ndone != 0) {
            fprintf(stderr, "emu: %d lanes left the kernel while others wait in a primitive\n", ndone);
            abort();
        }
        for (int l = 1; l < 64; ++l)
            if (g_tag[l] != g_tag[0] || g_nb[l] != g_nb[0]) {
                fprintf(stderr, "emu: lanes diverged at a primitive (lane %d tag %u vs lane 0 tag %u)\n", l, g_tag[l], g_tag[0]);
                abort();
            }
    }
}

}  // namespace emu

namespace estbe {

static std::string g_err;
const char *last_error() { return g_err.c_str(); }
int init() { return 0; }
void *dmalloc(size_t bytes) {
    void *p = nullptr;
    if (posix_memalign(&p, 256, bytes ? bytes : 256)) return nullptr;
    memset(p, 0xA5, bytes);  // uninitialised device memory is not zero
    return p;
}
void dfree(void *p) { free(p); }
size_t mem_free() { return (size_t)2 << 30; }
int h2d(void *d, const void *s, size_t n, void *) { if (n) memcpy(d, s, n); return 0; }
int d2h(void *d, const void *s, size_t n, void *) { if (n) memcpy(d, s, n); return 0; }
int d2d(void *d, const void *s, size_t n, void *) { if (n) memcpy(d, s, n); return 0; }
int zero(void *d, size_t n, void *) { if (n) memset(d, 0, n); return 0; }
int sync(void *) { return 0; }

int launch_cfg(const EstCfgArgs &a, void *) {
    for (uint32_t t = 0; t < 7; ++t) estdev::cfg_thread(a, t, 7);
    return 0;
}
int launch_prep1(const EstPrepArgs &a, void *) {
    for (uint32_t t = 0; t < 7; ++t) estdev::prep1_thread(a, t, 7);
    return 0;
}
int launch_prep2(const EstPrepArgs &a, void *) {
    for (uint32_t t = 0; t < 7; ++t) estdev::prep2_thread(a, t, 7);
    return 0;
}
int launch_envelope(const EstEnvArgs &a, void *) {
    for (uint64_t j = 0; j < a.n; j += a.per_wave)
        for (uint32_t i = 0; i < a.n_win; ++i)
            emu::run_wave([&] { estdev::envelope_wave(a, i, (uint32_t)j, (uint32_t)(j + a.per_wave < a.n ? j + a.per_wave : a.n)); });
    return 0;
}
// The wavefronts of all workgroups take turns, one step each, until every one has ended (a full turn in which nobody
// finds anything to do is a stuck candidate).
int launch_sim(const EstSimArgs &a, void *) {
    const uint32_t groups = (a.n_slots + a.per_group - 1) / a.per_group, total = groups * a.waves;
    const size_t words = (a.shared_bytes + (size_t)a.lds_bytes * a.waves) / 8 + 1;
    std::vector<std::vector<uint64_t>> lds(groups, std::vector<uint64_t>(words, 0x5A5A5A5A5A5A5A5Aull));
    std::vector<uint32_t> at(total, 0);
    std::vector<char> ended(total, 0);
    for (uint32_t g = 0; g < groups; ++g)
        emu::run_wave([&] { estdev::pool_setup(estdev::make_pool(a, (uint32_t *)lds[g].data())); });
    for (uint32_t left = total; left > 0;) {
        bool worked = false;
        for (uint32_t i = 0; i < total; ++i) {
            if (ended[i]) continue;
            const uint32_t g = i / a.waves, w = i % a.waves;
            uint64_t *mine = lds[g].data() + a.shared_bytes / 8 + (size_t)w * (a.lds_bytes / 8);
            uint32_t r = 0, next = at[i];
            emu::run_wave([&] {
                uint32_t my_at = at[i];
                const estdev::Pool p = estdev::make_pool(a, (uint32_t *)lds[g].data());
                const uint32_t x = a.skip_ops     ? estdev::pool_step<false, true>(p, g, w, my_at, mine)
                                   : a.dbg_ticks ? estdev::pool_step<true, false>(p, g, w, my_at, mine)
                                                 : estdev::pool_step<false, false>(p, g, w, my_at, mine);
                if (wv::lane() == 0) { r = x; next = my_at; }
            });
            at[i] = next;
            if (r == estdev::STEP_END) { ended[i] = 1; --left; }
            worked = worked || r != estdev::STEP_IDLE;
        }
        if (!worked) {
            a.status->sim_error = 1;
            break;
        }
    }
    return 0;
}
uint32_t max_resident_groups(uint32_t waves, uint32_t, uint32_t) { return waves <= 4 ? 2 : 0; }

void *stream_create() { return malloc(1); }  // everything runs in program order here
void stream_destroy(void *s) { free(s); }
int stream_wait_event(void *, void *) { return 0; }

void *static_scratch(uint64_t *bytes) {
    static std::vector<unsigned char> buf(EST_STATIC_SCRATCH_BYTES + 256);
    if (bytes) *bytes = EST_STATIC_SCRATCH_BYTES;
    return (void *)(((uintptr_t)buf.data() + 255) & ~(uintptr_t)255);
}
void *host_pinned_alloc(size_t bytes) { return malloc(bytes ? bytes : 1); }
void host_pinned_free(void *p) { free(p); }

void *event_create() { return malloc(1); }
void event_destroy(void *e) { free(e); }
int event_record(void *, void *) { return 0; }
float event_ms(void *, void *) { return 0.f; }

}  // namespace estbe
