// The C ABI (capi.cpp) built for the host over a stand-in for the HIP runtime and
// the kernels' launchers, all of whose calls end at once and any of which can be
// made to fail.  The launchers do what the kernels do to what capi.cpp keeps between
// calls: the sweep counter's words, the partial sums' places, the queues of launches
// that hold whole sweeps.  Usage: capi_host <scenario>; prints what went wrong
// and exits with 1, or nothing and 0.
#include <hip/hip_runtime.h>
#include <unistd.h>

#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <filesystem>
#include <map>
#include <string>
#include <vector>

#include "kernels.h"
#include "su3hb.h"

using namespace su3hb;

namespace {

int g_bad = 0;
std::map<char *, size_t> g_memory;   // device allocations
int g_fail_in = -1;                  // launches until one fails; -1: none
uint32_t g_swept = 0;                // last sweep index that a slice drew with
uint32_t g_slices = 0;               // slices done
bool g_give_up = false;              // launches of whole sweeps give up a wait
bool g_capturing = false;            // the stream is being captured
bool g_busy = false;                 // work that was there before runs on the stream
int g_polls = 0;                     // event queries meanwhile
size_t g_differ = 0;                 // doubles that a copy of links got wrong

void bad(const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vprintf(fmt, ap);
    va_end(ap);
    printf("\n");
    ++g_bad;
}

#define EXPECT(cond)                                                        \
    do {                                                                    \
        if (!(cond)) bad("line %d: not %s (%s)", __LINE__, #cond, su3hb_last_error()); \
    } while (0)

hipError_t launch() { return g_fail_in >= 0 && g_fail_in-- == 0 ? hipErrorUnknown : hipSuccess; }

bool in_memory(const void *p, size_t bytes)
{
    for (auto &m : g_memory)
        if (static_cast<const char *>(p) >= m.first && static_cast<const char *>(p) + bytes <= m.first + m.second)
            return true;
    return false;
}

int threads()
{
    int n = 0;
    for (const auto &f : std::filesystem::directory_iterator("/proc/self/task")) n += f.exists();
    return n;
}

// what a slice kernel does besides its links
hipError_t slice(int D, const UpdateArgs &a)
{
    if (hipError_t e = launch()) return e;
    const uint32_t sweep = a.sweep[a.parity];
    g_swept = sweep;
    ++g_slices;
    if (a.meas != nullptr && a.parity == 1) {
        double *m = a.meas + (size_t(a.sweep[3]) * D + a.mu) * a.total_blocks * a.meas_classes;
        const size_t n = size_t(a.total_blocks) * a.meas_classes;
        if (!in_memory(m, n * sizeof(double))) bad("partial sums of place %u outside their buffer", a.sweep[3]);
        else
            for (size_t i = 0; i < n; ++i) m[i] = sweep;
    }
    if (a.mu == D - 1) {  // advance_sweep
        a.sweep[1 - a.parity] = sweep + uint32_t(a.parity);
        if (a.meas != nullptr) a.sweep[3 - a.parity] = a.sweep[2 + a.parity] + uint32_t(a.parity);
    }
    return hipSuccess;
}

}  // namespace

// ---------------------------------------------------------------------------
// the runtime

extern "C" {

void **__hipRegisterFatBinary(const void *) { return nullptr; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}

hipError_t hipMalloc(void **p, size_t n)
{
    *p = std::calloc(n, 1);
    g_memory[static_cast<char *>(*p)] = n;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    g_memory.erase(static_cast<char *>(p));
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return (*p = std::calloc(n, 1)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "an error"; }
hipError_t hipGetSymbolAddress(void **, const void *) { return hipErrorInvalidSymbol; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *at, const void *)
{
    at->type = hipMemoryTypeUnregistered;
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s)
{
    *s = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t)
{
    if (g_capturing) bad("a captured stream is waited for");
    if (g_busy && threads() != 1) bad("%d threads while the stream is waited for", threads());
    g_busy = false;
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = reinterpret_cast<hipEvent_t>(1); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t)
{
    if (!g_busy) return hipSuccess;
    usleep(100);
    if (++g_polls < 100) return hipErrorNotReady;
    bad("%d threads poll while earlier work runs", threads());
    g_busy = false;
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }

}  // extern "C"

// ---------------------------------------------------------------------------
// the launchers

namespace su3hb {

hipError_t launch_update(int D, int, int, dim3, dim3, hipStream_t, const UpdateArgs &a) { return slice(D, a); }
hipError_t launch_update_split(int D, int, hipStream_t, const UpdateArgs &a) { return slice(D, a); }
hipError_t launch_update_planes(int D, int, hipStream_t, const UpdateArgs &a) { return slice(D, a); }
hipError_t launch_update_small(int D, int, hipStream_t, const SmallArgs &s)
{
    if (hipError_t e = launch()) return e;
    if (s.work[kSmallTicket] != 0) {
        bad("a queue that is not empty: no sweep is done");
        return hipSuccess;
    }
    s.work[kSmallTicket] = s.items + 1;
    if (g_give_up) {
        *s.failed = 1;
        return hipSuccess;
    }
    g_swept = s.sweep0 + s.sweeps - 1;
    g_slices += 2u * uint32_t(D) * s.sweeps;
    s.u.sweep[0] = s.sweep0 + s.sweeps;
    if (s.u.meas)
        for (uint32_t i = 0; i < s.sweeps; ++i) s.series[6 * i] = s.sweep0 + i;
    return hipSuccess;
}
hipError_t launch_update_persistent(int, int, int, hipStream_t, const UpdateArgs &a, int n)
{
    if (hipError_t e = launch()) return e;
    g_swept = a.sweep[0] + uint32_t(n) - 1;
    return hipSuccess;
}
hipError_t persistent_max_blocks(int, int, int *n) { *n = 2; return hipSuccess; }
hipError_t update_lds(int, int, int, dim3, const UpdateArgs &, size_t *need, size_t *limit)
{
    *need = 0;
    *limit = 1;
    return hipSuccess;
}
hipError_t launch_plaquette(int, int, dim3, dim3, hipStream_t, const PlaqArgs &) { return launch(); }
hipError_t launch_plaquette_finalize(hipStream_t, const RepDesc *, int, int, const double *, double *) { return launch(); }
hipError_t launch_measure_finalize(hipStream_t, const double *meas, int n, int D, uint32_t nblocks, int nc, double, int,
                                   double, double, double *series, uint32_t *sweep)
{
    if (hipError_t e = launch()) return e;
    if (sweep[2] != uint32_t(n)) bad("%u measured sweeps wait, %d are added up", sweep[2], n);
    for (int i = 0; i < n; ++i) series[6 * i] = meas[(size_t(i) * D + 1) * nblocks * nc];
    sweep[2] = 0;
    return hipSuccess;
}
hipError_t launch_start(int, int, hipStream_t, void *, const RepDesc *, int, uint32_t, int) { return launch(); }
// element i of the canonical links is i
hipError_t launch_pack(int D, int, hipStream_t, const void *, const RepDesc *, int, uint64_t c0, uint32_t count, double *dst)
{
    if (hipError_t e = launch()) return e;
    for (size_t i = 0, n = size_t(D) * 18; i < count * n; ++i) dst[i] = double(c0 * n + i);
    return hipSuccess;
}
hipError_t launch_unpack(int D, int, hipStream_t, void *, const RepDesc *, int, uint64_t c0, uint32_t count, const double *src)
{
    if (hipError_t e = launch()) return e;
    for (size_t i = 0, n = size_t(D) * 18; i < count * n; ++i) g_differ += src[i] != double(c0 * n + i);
    return hipSuccess;
}
hipError_t launch_validate(hipStream_t, const double *, uint64_t, unsigned long long *) { return launch(); }
hipError_t launch_rep_set(hipStream_t, const RepDesc &r, RepDesc *d) { *d = r; return launch(); }
hipError_t launch_stats_zero(hipStream_t, StatSlot *) { return launch(); }
hipError_t launch_stats_reduce(hipStream_t, StatSlot *, StatSlot *) { return launch(); }
hipError_t launch_counter_add(hipStream_t, uint32_t *c, uint32_t n) { if (hipError_t e = launch()) return e; *c += n; return hipSuccess; }
hipError_t launch_counter_set(hipStream_t, uint32_t *c, uint32_t v) { if (hipError_t e = launch()) return e; *c = v; return hipSuccess; }
hipError_t launch_measure_begin(hipStream_t, uint32_t *s) { if (hipError_t e = launch()) return e; s[2] = 0; return hipSuccess; }
hipError_t launch_u32_zero(hipStream_t, uint32_t *p, int n)
{
    if (hipError_t e = launch()) return e;
    for (int i = 0; i < n; ++i) p[i] = 0;
    return hipSuccess;
}
hipError_t launch_u64_zero(hipStream_t, unsigned long long *p, int n)
{
    if (hipError_t e = launch()) return e;
    for (int i = 0; i < n; ++i) p[i] = 0;
    return hipSuccess;
}

}  // namespace su3hb

// ---------------------------------------------------------------------------

namespace {

su3hb_lattice *lattice(std::vector<int> ext, void *stream = nullptr)
{
    su3hb_params p{};
    p.nd = int(ext.size());
    for (size_t i = 0; i < ext.size(); ++i) p.extents[i] = ext[i];
    p.nlat = 1;
    p.start = SU3HB_COLD;
    p.seed = 1;
    p.hip_stream = stream;
    su3hb_lattice *L = nullptr;
    if (su3hb_init_lattice(&L, &p) != SU3HB_OK) {
        bad("no lattice: %s", su3hb_last_error());
        std::exit(1);
    }
    return L;
}

uint64_t sweep_of(const su3hb_lattice *L)
{
    uint64_t n = 0;
    su3hb_get_state(L, nullptr, &n);
    return n;
}

// A call of 3 measured sweeps fails at its k-th launch, for every k; the next call,
// which fills the room of the partial sums, keeps to it, gives its own rows and
// draws with the sweep indices that the handle counts.
void failed_measurement()
{
    for (const std::vector<int> &ext : {std::vector<int>{4, 4}, {12, 8, 8, 6}, {16, 16, 16, 16}, {24, 24, 24, 16}})
        for (int timed = 0; timed < 2; ++timed)
            for (int k = 0;; ++k) {
                su3hb_lattice *L = lattice(ext);
                double series[6 * 16] = {}, timing[4];
                EXPECT(su3hb_sweep(L, 6, 6, 8, 2, nullptr) == SU3HB_OK);
                g_fail_in = k;
                const int rc = timed ? su3hb_sweep_timed(L, 6, 6, 8, 3, 1, series, timing)
                                     : su3hb_sweep_measure(L, 6, 6, 8, 3, series, nullptr);
                const bool failed = g_fail_in < 0;
                g_fail_in = -1;
                EXPECT(rc == (failed ? SU3HB_EHIP : SU3HB_OK));
                const uint64_t at = sweep_of(L);
                EXPECT(su3hb_sweep_measure(L, 6, 6, 8, 16, series, nullptr) == SU3HB_OK);
                for (int i = 0; i < 16; ++i) EXPECT(series[6 * i] == double(at + uint64_t(i)));
                EXPECT(g_swept == at + 15 && sweep_of(L) == at + 16);
                su3hb_free(L);
                if (!failed) break;
            }
}

// A call of unmeasured sweeps that fails between its launches leaves the sweep
// indices of later ones as the handle counts them.
void failed_sweeps()
{
    for (const std::vector<int> &ext : {std::vector<int>{4, 4}, {12, 8, 8, 6}, {24, 24, 24, 16}})
        for (int k = 0;; ++k) {
            su3hb_lattice *L = lattice(ext);
            EXPECT(su3hb_sweep(L, 6, 6, 8, 2, nullptr) == SU3HB_OK);
            g_fail_in = k;
            su3hb_stats st;
            const int rc = su3hb_sweep(L, 6, 6, 8, 3, k % 2 ? &st : nullptr);
            const bool failed = g_fail_in < 0;
            g_fail_in = -1;
            EXPECT(rc == (failed ? SU3HB_EHIP : SU3HB_OK));
            const uint64_t at = sweep_of(L);
            EXPECT(su3hb_sweep(L, 6, 6, 8, 1, nullptr) == SU3HB_OK);
            EXPECT(g_swept == at);
            su3hb_free(L);
            if (!failed) break;
        }
    // a batch, slice by slice and in persistent launches
    su3hb_replica_desc reps[2] = {};
    for (auto &r : reps) {
        for (int i = 0; i < 4; ++i) r.extents[i] = 8;
        r.beta = 6;
        r.start = SU3HB_COLD;
    }
    for (int mode = 0; mode < 2; ++mode)
        for (int k = 0;; ++k) {
            su3hb_batch *B = nullptr;
            EXPECT(su3hb_batch_create(&B, 4, reps, 2, SU3HB_FP64_18, nullptr) == SU3HB_OK);
            EXPECT(su3hb_batch_sweep(B, 8, 2, 0, nullptr) == SU3HB_OK);
            g_fail_in = k;
            const int rc = su3hb_batch_sweep(B, 8, 3, mode, nullptr);
            const bool failed = g_fail_in < 0;
            g_fail_in = -1;
            EXPECT(rc == (failed ? SU3HB_EHIP : SU3HB_OK));
            const uint64_t at = sweep_of(B);
            EXPECT(su3hb_batch_sweep(B, 8, 1, 1 - mode, nullptr) == SU3HB_OK);
            EXPECT(g_swept == at);
            su3hb_batch_free(B);
            if (!failed) break;
        }
}

// A launch of whole sweeps gives up a wait.  Every call that synchronises says so,
// until set_links has replaced the links (of every replica); then all is as the
// handle counts it.
void given_up_waits()
{
    std::vector<double> links;
    double series[6 * 4], out[6], timing[4];
    su3hb_stats st;
    using Call = int (*)(su3hb_lattice *, double *, double *, double *, su3hb_stats *, std::vector<double> &);
    const Call calls[] = {
        [](su3hb_lattice *L, double *, double *o, double *, su3hb_stats *, std::vector<double> &) { return su3hb_plaquette(L, 6, 6, o); },
        [](su3hb_lattice *L, double *, double *, double *, su3hb_stats *, std::vector<double> &l) { return su3hb_get_links(L, l.data(), l.size()); },
        [](su3hb_lattice *L, double *, double *, double *, su3hb_stats *s, std::vector<double> &) { return su3hb_sweep(L, 6, 6, 8, 1, s); },
        [](su3hb_lattice *L, double *, double *, double *, su3hb_stats *s, std::vector<double> &) { return su3hb_overrelax(L, 6, 6, 1, s); },
        [](su3hb_lattice *L, double *s, double *, double *, su3hb_stats *, std::vector<double> &) { return su3hb_sweep_measure(L, 6, 6, 8, 4, s, nullptr); },
        [](su3hb_lattice *L, double *s, double *, double *t, su3hb_stats *, std::vector<double> &) { return su3hb_sweep_timed(L, 6, 6, 8, 2, 1, s, t); },
        [](su3hb_lattice *L, double *, double *, double *, su3hb_stats *, std::vector<double> &) { return su3hb_set_launch(L, 256, 1, 2); },
        [](su3hb_lattice *L, double *, double *, double *, su3hb_stats *, std::vector<double> &) { return su3hb_autotune(L, 1); },
    };
    for (size_t c = 0; c < sizeof calls / sizeof *calls; ++c) {
        const int n1 = 4 + 2 * int(c);  // shapes that nothing has tuned
        su3hb_lattice *L = lattice({4, n1});
        links.assign(size_t(4 * n1 * 2 * 18), 0.0);
        g_give_up = true;
        EXPECT(su3hb_sweep(L, 6, 6, 8, 3, nullptr) == SU3HB_OK);
        g_give_up = false;
        for (int twice = 0; twice < 2; ++twice) {
            const int rc = calls[c](L, series, out, timing, &st, links);
            if (rc != SU3HB_EHIP) bad("call %zu returns %d", c, rc);
        }
        EXPECT(su3hb_set_state(L, 1, 7) == SU3HB_OK);
        EXPECT(su3hb_plaquette(L, 6, 6, out) == SU3HB_EHIP);
        EXPECT(su3hb_set_links(L, links.data(), links.size()) == SU3HB_OK);
        for (size_t k = 0; k < sizeof calls / sizeof *calls; ++k) {
            const int rc = calls[k](L, series, out, timing, &st, links);
            if (rc != SU3HB_OK) bad("after set_links call %zu returns %d (%s)", k, rc, su3hb_last_error());
        }
        const uint64_t at = sweep_of(L);
        EXPECT(at == 7 + 1 + 1 + 4 + 2);
        EXPECT(su3hb_sweep_timed(L, 6, 6, 8, 1, 0, nullptr, timing) == SU3HB_OK && g_swept == at);
        su3hb_free(L);
    }
    // the sweep index of a launch that did not step the device's
    su3hb_lattice *L = lattice({4, 40});
    links.assign(4 * 40 * 2 * 18, 0.0);
    g_give_up = true;
    EXPECT(su3hb_sweep(L, 6, 6, 8, 3, nullptr) == SU3HB_OK);
    g_give_up = false;
    EXPECT(su3hb_set_links(L, links.data(), links.size()) == SU3HB_OK);
    EXPECT(su3hb_sweep_timed(L, 6, 6, 8, 1, 0, nullptr, timing) == SU3HB_OK);
    EXPECT(g_swept == 3 && sweep_of(L) == 4);
    su3hb_free(L);

    su3hb_replica_desc reps[3] = {};
    for (auto &r : reps) {
        r.extents[0] = r.extents[1] = 4;
        r.beta = 6;
        r.start = SU3HB_COLD;
    }
    su3hb_batch *B = nullptr;
    EXPECT(su3hb_batch_create(&B, 2, reps, 3, SU3HB_FP64_18, nullptr) == SU3HB_OK);
    std::vector<double> rows(18);
    const size_t n = 4 * 4 * 2 * 18;
    g_give_up = true;
    EXPECT(su3hb_batch_sweep(B, 8, 2, 0, nullptr) == SU3HB_OK);
    g_give_up = false;
    EXPECT(su3hb_batch_sweep(B, 8, 1, 1, nullptr) == SU3HB_EHIP);
    EXPECT(su3hb_batch_plaquette(B, rows.data(), rows.size()) == SU3HB_EHIP);
    EXPECT(su3hb_batch_get_links(B, 1, links.data(), n) == SU3HB_EHIP);
    for (int r : {0, 1}) EXPECT(su3hb_batch_set_links(B, r, links.data(), n) == SU3HB_OK);
    EXPECT(su3hb_batch_sweep(B, 8, 1, 0, nullptr) == SU3HB_OK);  // all replicas in doubt again
    for (int r : {2, 0, 1}) {
        EXPECT(su3hb_batch_plaquette(B, rows.data(), rows.size()) == SU3HB_EHIP);
        EXPECT(su3hb_batch_set_links(B, r, links.data(), n) == SU3HB_OK);
    }
    EXPECT(su3hb_batch_plaquette(B, rows.data(), rows.size()) == SU3HB_OK);
    EXPECT(su3hb_batch_sweep(B, 8, 1, 1, nullptr) == SU3HB_OK);
    su3hb_batch_free(B);
}

// More calls than there are queues, of which one fails at its first, second or
// third launch: no later one gets a queue that has been used.
void failed_clearing()
{
    for (int k = 0; k < 3; ++k)
        for (uint32_t nth : {0u, 1u, kSmallQueues - 1, kSmallQueues, kSmallQueues + 1}) {
            su3hb_lattice *L = lattice({4, 4});
            for (uint32_t i = 0; i < 3 * kSmallQueues; ++i) {
                if (i == nth || i == nth + kSmallQueues) g_fail_in = k;
                const int rc = su3hb_sweep(L, 6, 6, 8, 1, nullptr);
                const bool failed = (i == nth || i == nth + kSmallQueues) && g_fail_in < 0;
                g_fail_in = -1;
                EXPECT(rc == (failed ? SU3HB_EHIP : SU3HB_OK));
                if (rc == SU3HB_OK) EXPECT(g_swept + 1 == sweep_of(L));
            }
            su3hb_free(L);
        }
}

// Large copies of links behind sweeps that still run: no thread is started before
// the sweeps have ended.
void copies_behind_sweeps()
{
    for (const std::vector<int> &ext : {std::vector<int>{8, 8, 8, 16}, {16, 16, 16, 16}, {16, 16, 30, 66}}) {
        static int stream;  // not the null stream, which cannot be captured
        su3hb_lattice *L = lattice(ext, &stream);
        size_t n = 4 * 18;
        for (int e : ext) n *= size_t(e);
        std::vector<double> links(n, -1.0);
        EXPECT(su3hb_sweep(L, 6, 6, 8, 1, nullptr) == SU3HB_OK);
        g_busy = true;
        g_polls = 0;
        EXPECT(su3hb_get_links(L, links.data(), n) == SU3HB_OK);
        size_t differ = 0;
        for (size_t i = 0; i < n; ++i) differ += links[i] != double(i);
        EXPECT(differ == 0 && !g_busy);
        g_busy = true;
        g_polls = 0;
        g_differ = 0;
        EXPECT(su3hb_set_links(L, links.data(), n) == SU3HB_OK);
        EXPECT(g_differ == 0 && !g_busy);
        // a captured stream is refused without a wait, which would end the capture
        g_capturing = true;
        EXPECT(su3hb_get_links(L, links.data(), n) == SU3HB_EHIP);
        if (n * sizeof(double) >= size_t(32) << 20) EXPECT(su3hb_set_links(L, links.data(), n) == SU3HB_EHIP);
        g_capturing = false;
        su3hb_free(L);
    }
}

}  // namespace

int main(int argc, char **argv)
{
    const std::map<std::string, void (*)()> scenarios = {
        {"failed_measurement", failed_measurement},
        {"failed_sweeps", failed_sweeps},
        {"given_up_waits", given_up_waits},
        {"failed_clearing", failed_clearing},
        {"copies_behind_sweeps", copies_behind_sweeps},
    };
    const auto it = argc == 2 ? scenarios.find(argv[1]) : scenarios.end();
    if (it == scenarios.end()) return 2;
    it->second();
    return g_bad ? 1 : 0;
}
