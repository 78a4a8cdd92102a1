// Host back end for the lock-step wavefront emulation (test infrastructure): "device" memory is
// host memory, a wavefront is 64 fibers that meet at every primitive.
//
// The wavefronts of a simulation launch are alive together, as on the device, and take turns.  EST_EMU_SCHEDULE unset: a
// wavefront keeps its turn for one whole step of the driver, so every operation runs from entry to exit undisturbed.
// EST_EMU_SCHEDULE=<seed>: a turn lasts a random number of primitives, from one to some hundred thousand, so that operations of
// the same candidate run inside one another and a wavefront may sleep anywhere while the others finish whole candidates.
// EST_EMU_WAVES: wavefronts of a workgroup at most (4 when unset).  EST_EMU_STILL_LIMIT: the driver's own limit on looks that find
// nothing, instead of the scheduler's knowledge of who is stuck.  EST_EMU_HOLD_LOCK: every candidate's last operation is locked by
// nobody, so that it never ends.
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>
#include <ucontext.h>

#include <functional>
#include <memory>
#include <random>
#include <string>
#include <vector>

#include "wave_emu.h"
#include "../../paper_1812_01776_amd/csrc/est_backend.h"
#include "../../paper_1812_01776_amd/csrc/est_device.h"

namespace emu {

namespace {
const size_t STACK = 128 * 1024;
const uint32_t TAG_TURN = 100;  // the rendezvous of a wavefront that gives up its turn

struct Wave {
    ucontext_t ctx[64];
    char *stacks;
    bool done[64];
    uint64_t x[2][64];
    uint32_t tag[64], nb[64];
    std::function<void()> body;
    Wave() {
        void *p = mmap(nullptr, 64 * STACK, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
        if (p == MAP_FAILED) abort();
        stacks = (char *)p;
    }
    ~Wave() { munmap(stacks, 64 * STACK); }
    Wave(const Wave &) = delete;
    Wave &operator=(const Wave &) = delete;
};

ucontext_t g_sched;
Wave *g_wave;
uint32_t g_cur;

void trampoline() {
    g_wave->body();
    g_wave->done[g_cur] = true;
    swapcontext(&g_wave->ctx[g_cur], &g_sched);
}

void start(Wave &w, const std::function<void()> &body) {
    w.body = body;
    for (int l = 0; l < 64; ++l) {
        w.done[l] = false;
        w.nb[l] = 0;
        getcontext(&w.ctx[l]);
        w.ctx[l].uc_stack.ss_sp = w.stacks + (size_t)l * STACK;
        w.ctx[l].uc_stack.ss_size = STACK;
        w.ctx[l].uc_link = &g_sched;
        makecontext(&w.ctx[l], trampoline, 0);
    }
}

// All lanes go on to the next primitive: its tag, or 0 when the wavefront has ended.
uint32_t advance(Wave &w) {
    g_wave = &w;
    int ndone = 0;
    for (int l = 0; l < 64; ++l) {
        if (w.done[l]) { ++ndone; continue; }
        g_cur = (uint32_t)l;
        swapcontext(&g_sched, &w.ctx[l]);
        if (w.done[l]) ++ndone;
    }
    if (ndone == 64) return 0;
    if (ndone != 0) {
        fprintf(stderr, "emu: %d lanes left the kernel while others wait in a primitive\n", ndone);
        abort();
    }
    for (int l = 1; l < 64; ++l)
        if (w.tag[l] != w.tag[0] || w.nb[l] != w.nb[0]) {
            fprintf(stderr, "emu: lanes 0 and %d are in different primitives (%u vs %u)\n", l, w.tag[0], w.tag[l]);
            abort();
        }
    return w.tag[0];
}
}  // namespace

uint32_t lane() { return g_cur; }

const uint64_t *exchange(uint64_t v, uint32_t tag) {
    Wave &w = *g_wave;
    const uint32_t me = g_cur;
    const uint32_t ph = w.nb[me] & 1u;
    w.x[ph][me] = v;
    w.tag[me] = tag;
    w.nb[me]++;
    swapcontext(&w.ctx[me], &g_sched);  // wait for the other lanes
    g_wave = &w;
    g_cur = me;
    return w.x[ph];
}

// One wavefront from start to end.
void run_wave(const std::function<void()> &body) {
    static Wave w;
    start(w, body);
    while (advance(w) != 0) {}
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
// what the launch would be, for a test of its size
extern "C" uint32_t emu_envelope_launch(uint64_t n, uint32_t n_win, uint32_t *per_wave) {
    *per_wave = envelope_per_wave(n, n_win);
    return envelope_groups(n, n_win, *per_wave);
}
int launch_envelope(const EstEnvArgs &a, void *) {
    for (uint64_t j = 0; j < a.n; j += a.per_wave)
        for (uint32_t i = 0; i < a.n_win; ++i)
            emu::run_wave([&] { estdev::envelope_wave(a, i, (uint32_t)j, (uint32_t)(j + a.per_wave < a.n ? j + a.per_wave : a.n)); });
    return 0;
}
// Every wavefront runs the driver's loop until it ends; when all that are left have found nothing to do since anybody last
// did something, a candidate is stuck.
int launch_sim(const EstSimArgs &a, void *) {
    const uint32_t groups = (a.n_slots + a.per_group - 1) / a.per_group, total = groups * a.waves;
    const size_t words = (a.shared_bytes + (size_t)a.lds_bytes * a.waves) / 8 + 1;
    std::vector<std::vector<uint64_t>> lds(groups, std::vector<uint64_t>(words, 0x5A5A5A5A5A5A5A5Aull));
    for (uint32_t g = 0; g < groups; ++g)
        emu::run_wave([&] { estdev::pool_setup(estdev::make_pool(a, (uint32_t *)lds[g].data())); });
    static std::vector<std::unique_ptr<emu::Wave>> pool;
    while (pool.size() < total) pool.emplace_back(new emu::Wave);
    const char *limit_env = getenv("EST_EMU_STILL_LIMIT");
    const uint32_t limit = limit_env ? (uint32_t)atol(limit_env) : ~0u;
    std::vector<char> quiet(total, 0);  // found nothing to do in a look that began after anybody last did something
    uint32_t events = 0;
    for (uint32_t i = 0; i < total; ++i) {
        const uint32_t g = i / a.waves, w = i % a.waves;
        uint64_t *mine = lds[g].data() + a.shared_bytes / 8 + (size_t)w * (a.lds_bytes / 8);
        emu::start(*pool[i], [&a, &lds, &quiet, &events, limit, g, w, i, mine] {
            const estdev::Pool p = estdev::make_pool(a, (uint32_t *)lds[g].data());
            uint32_t at = 0;
            estdev::Wait wait = {0, 0, 0};
            for (;;) {
                const uint32_t before = events;
                quiet[i] = 0;
                const uint32_t r = a.skip_ops     ? estdev::pool_step<false, true>(p, g, w, at, mine)
                                   : a.dbg_ticks ? estdev::pool_step<true, false>(p, g, w, at, mine)
                                                 : estdev::pool_step<false, false>(p, g, w, at, mine);
                if (wv::lane() == 0) {
                    if (r == estdev::STEP_IDLE) {
                        quiet[i] = events == before;
                    } else {
                        ++events;
                        quiet.assign(quiet.size(), 0);
                    }
                }
                if (r == estdev::STEP_END) break;
                if (r == estdev::STEP_IDLE && (estdev::stuck(p, wait, limit) || wv::uniform(a.status->sim_error))) {
                    a.status->sim_error = 1;
                    break;
                }
                (void)emu::exchange(0, emu::TAG_TURN);
            }
        });
    }
    const char *seed = getenv("EST_EMU_SCHEDULE");
    std::mt19937_64 rng(seed ? (uint64_t)atoll(seed) : 0);
    std::vector<char> ended(total, 0);
    const uint32_t top = 6 + (uint32_t)(rng() % 12);
    const bool hold = getenv("EST_EMU_HOLD_LOCK") != nullptr;
    for (uint32_t left = total, turn = 0; left > 0; ++turn) {
        for (uint32_t g = 0; g < groups && hold; ++g) {
            uint32_t *ctl = estdev::slot_ctl(estdev::make_pool(a, (uint32_t *)lds[g].data()), 0);
            if (ctl[estdev::C_PHASE] == estdev::PH_RUN && ctl[estdev::C_LOCK + a.n_ops - 1] == 0) ctl[estdev::C_LOCK + a.n_ops - 1] = 1;
        }
        const uint32_t i = seed ? (uint32_t)(rng() % total) : turn % total;
        if (ended[i]) continue;
        uint64_t length = seed ? 1ull << (rng() % top) : ~0ull;
        uint32_t tag = 1;
        while (length-- > 0 && (tag = emu::advance(*pool[i])) != 0 && tag != emu::TAG_TURN) {}
        if (tag == 0) { ended[i] = 1; --left; }
        bool stuck = left > 0 && !limit_env;
        for (uint32_t k = 0; k < total && stuck; ++k) stuck = ended[k] || quiet[k];
        if (stuck) {
            a.status->sim_error = 1;
            break;
        }
    }
    return 0;
}
// (two workgroups at a time: what the launches of one call share is in play)
uint32_t max_resident_groups(uint32_t waves, uint32_t, uint32_t) {
    const char *most = getenv("EST_EMU_WAVES");
    return waves <= (most ? (uint32_t)atoi(most) : 4u) ? 2 : 0;
}

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
