// A model of the HIP calls that the block cache (devmem.hip) makes, and
// scenarios over it: streams are vector clocks, so that every use of a block
// can be checked to come after the uses before it, whatever a GPU's timing.
// All streams but the null stream are non-blocking here, the weakest order
// that a caller may have.  Usage: <program> <scenario>; prints what went wrong.
#include <algorithm>
#include <array>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "devmem.hip"

namespace idx {
int hip_fail(hipError_t) { return IDX_ERR_HIP; }
}  // namespace idx

namespace {

constexpr int kStreams = 4;
using Clock = std::array<uint64_t, kStreams>;
char g_handle[kStreams];
const hipStream_t S0 = nullptr, SA = (hipStream_t)&g_handle[1], SB = (hipStream_t)&g_handle[2],
                  SC = (hipStream_t)&g_handle[3];  // SC: the stream that a scenario captures
Clock g_clock[kStreams];
Clock g_host;  // what the host has waited for

struct Mem {
    size_t bytes;
    bool live;
    Clock used;  // its last use, or its free
};
std::map<char *, Mem> g_mem;
size_t g_held = 0, g_capacity = ~(size_t)0;  // live, and freed but still in the pool
char *g_next = (char *)0x100000;
std::map<hipEvent_t, Clock> g_events;
uint64_t g_event_id = 0;
bool g_no_wait = false;  // waits for events and for the device fail
bool g_capture = false;  // SC is being captured (a blocking stream, any thread)
std::vector<std::string> g_wrong;

void wrong(const std::string &what) {
    if (g_wrong.size() < 5) g_wrong.push_back(what);
}
int g_dev = 0;  // current device; device 1 has a null stream alone, with SC's clock
int id(hipStream_t s) { return s == nullptr ? 3 * g_dev : (int)((char *)s - g_handle); }
bool before(const Clock &a, const Clock &b) {
    for (int i = 0; i < kStreams; ++i)
        if (a[i] > b[i]) return false;
    return true;
}
void join(Clock &a, const Clock &b) {
    for (int i = 0; i < kStreams; ++i) a[i] = std::max(a[i], b[i]);
}
Clock op(hipStream_t s) {
    Clock &c = g_clock[id(s)];
    ++c[id(s)];
    return c;
}
// Work on the null stream (or the device) while a blocking stream is captured.
bool breaks_capture(hipStream_t s, const char *call) {
    if (s != nullptr || !g_capture) return false;
    wrong(std::string(call) + " on the null stream during another stream's capture");
    return true;
}

void use(void *p, hipStream_t s) {
    auto it = g_mem.find((char *)p);
    if (it == g_mem.end() || !it->second.live) return wrong("use of memory that is not live");
    if (!before(it->second.used, g_clock[id(s)])) wrong("a block's use is not ordered after the one before it");
    it->second.used = op(s);
}

}  // namespace

extern "C" {
hipError_t hipGetDevice(int *d) { *d = g_dev; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipDeviceGetDefaultMemPool(hipMemPool_t *p, int) { *p = nullptr; return hipSuccess; }
hipError_t hipMemPoolSetAttribute(hipMemPool_t, hipMemPoolAttr, void *) { return hipSuccess; }
hipError_t hipMemPoolTrimTo(hipMemPool_t, size_t) {  // freed blocks that the host has waited for
    for (auto &m : g_mem)
        if (!m.second.live && m.second.bytes && before(m.second.used, g_host)) {
            g_held -= m.second.bytes;
            m.second.bytes = 0;
        }
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *st) {
    *st = s == SC && g_capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return s == nullptr && g_capture ? hipErrorStreamCaptureImplicit : hipSuccess;
}
hipError_t hipMallocAsync(void **p, size_t bytes, hipStream_t s) {
    if (breaks_capture(s, "hipMallocAsync")) return hipErrorStreamCaptureImplicit;
    if (bytes > g_capacity || g_held > g_capacity - bytes) return hipErrorOutOfMemory;
    g_held += bytes;
    g_mem[g_next] = Mem{bytes, true, op(s)};
    *p = g_next;
    g_next += (bytes + 255) / 256 * 256 + 256;
    return hipSuccess;
}
hipError_t hipFreeAsync(void *p, hipStream_t s) {
    if (breaks_capture(s, "hipFreeAsync")) return hipErrorStreamCaptureImplicit;
    use(p, s);
    g_mem[(char *)p].live = false;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    *e = (hipEvent_t)(uintptr_t)++g_event_id;
    g_events[*e] = Clock{};
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
    if (!g_events.erase(e)) wrong("an event destroyed twice");
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    if (breaks_capture(s, "hipEventRecord")) return hipErrorStreamCaptureImplicit;
    g_events[e] = op(s);
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    if (breaks_capture(s, "hipStreamWaitEvent")) return hipErrorStreamCaptureImplicit;
    if (g_no_wait) return hipErrorUnknown;
    join(g_clock[id(s)], g_events[e]);
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
    if (g_no_wait) return hipErrorUnknown;
    join(g_host, g_events[e]);
    for (auto &c : g_clock) join(c, g_host);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
    if (breaks_capture(s, "hipStreamSynchronize")) return hipErrorStreamCaptureImplicit;
    join(g_host, g_clock[id(s)]);
    return hipSuccess;
}
hipError_t hipDeviceSynchronize(void) {
    if (breaks_capture(nullptr, "hipDeviceSynchronize")) return hipErrorStreamCaptureImplicit;
    if (g_no_wait) return hipErrorUnknown;
    for (auto &c : g_clock) join(g_host, c);
    for (auto &c : g_clock) join(c, g_host);
    return hipSuccess;
}
}

namespace {

constexpr size_t MiB = 1 << 20;

void *get(size_t bytes, hipStream_t s) {
    hipError_t e = hipSuccess;
    void *p = idx::cached_get(bytes, s, &e);
    if (p) use(p, s);
    return p;
}

void put(void *p, hipStream_t s) { idx::cached_put(p, s); }

// Blocks of changing sizes pass between the null stream and two others, freed
// while still in use there; more requests than an idle block outlives.
void order() {
    srand(7);
    const hipStream_t all[3] = {S0, SA, SB};
    struct Held { void *p; hipStream_t s; };
    std::vector<Held> held;
    for (int i = 0; i < 20000; ++i) {
        if (held.size() < 12 && (held.empty() || rand() % 2)) {
            const hipStream_t s = all[rand() % 3];
            void *p = get((size_t)(1 + rand() % 8) * (rand() % 8 ? MiB : 900 * MiB), s);
            if (!p) return wrong("no memory");
            held.push_back({p, s});
        } else {
            const size_t j = rand() % held.size();
            use(held[j].p, held[j].s);
            put(held[j].p, held[j].s);
            held.erase(held.begin() + j);
        }
        size_t live = 0, n = 0;  // handed out and idle
        for (auto &m : g_mem)
            if (m.second.live) {
                live += m.second.bytes;
                ++n;
            }
        for (auto &h : held) live -= g_mem[(char *)h.p].bytes;
        if (live > 2 * (8ull << 30) || n - held.size() > 2 * 256) return wrong("more idle memory than the cache's bounds");
    }
}

// Blocks freed on the null stream, wanted or pushed out by another stream's
// calls while a third stream is captured.
void capture_elsewhere() {
    put(get(3 * MiB, S0), S0);
    for (int i = 0; i < 8; ++i) put(get(1000 * MiB + i * 30 * MiB, S0), S0);
    g_capture = true;
    void *p = get(3 * MiB, SA);
    if (!p) return wrong("no memory");
    put(p, SA);
    for (int i = 0; i < 600; ++i) {
        void *a = get((size_t)(1 + i % 40) * 40 * MiB, SA);
        if (!a) return wrong("no memory");
        put(a, SA);
    }
    // the captured stream's own blocks are graph nodes
    void *c = get(3 * MiB, SC);
    put(c, SC);
    g_capture = false;
    if (!c || g_mem[(char *)c].live) wrong("a captured stream's block stayed in the cache");
}

// A block whose last use cannot be waited for is neither handed out nor freed;
// it serves again once it can be.
void failed_wait() {
    void *p = get(3 * MiB, SA);
    use(p, SA);
    put(p, SA);
    g_no_wait = true;
    void *q = get(3 * MiB, SB);
    if (!q || q == p) return wrong("a block was handed out unordered");
    for (int i = 0; i < 600; ++i) put(get((size_t)(1 + i % 40) * 40 * MiB, SB), SB);  // outlives and pushes out
    g_no_wait = false;
    if (get(3 * MiB, SA) != p) wrong("the block was lost");
}

// A request that does not fit beside the idle blocks gets their memory, also
// one larger than the cache keeps, and also from the null stream's blocks.
void memory_short() {
    g_capacity = 12ull << 30;
    const size_t sizes[] = {7ull << 30, 11ull << 30};
    const hipStream_t from[] = {S0, SA}, to[] = {S0, SA, SB};
    for (size_t bytes : sizes)
        for (hipStream_t f : from)
            for (hipStream_t t : to) {
                std::vector<void *> p;
                for (int i = 0; i < 6; ++i) p.push_back(get((900 + 10 * i) * MiB, f));
                for (void *q : p) {
                    if (!q) return wrong("no memory for the first blocks");
                    use(q, f);
                    put(q, f);
                }
                void *big = get(bytes, t);
                if (!big) return wrong("no memory, with idle blocks kept");
                put(big, t);
                (void)hipStreamSynchronize(t);  // one larger than the cache keeps is freed
            }
    // what the null stream freed stays out of reach during another stream's capture
    void *p = get(7ull << 30, S0);
    if (!p) return wrong("no memory");
    put(p, S0);
    g_capture = true;
    if (get(8ull << 30, SA)) wrong("memory from nowhere");
    g_capture = false;
    if (!get(8ull << 30, SA)) wrong("no memory after the capture");
}

// Every idle block goes back on request, whichever stream freed it.
void trim() {
    const hipStream_t all[3] = {S0, SA, SB};
    void *kept = get(5 * MiB, SB);
    for (int i = 0; i < 30; ++i) put(get((size_t)(1 + i) * 7 * MiB, all[i % 3]), all[i % 3]);
    if (idx::cached_trim() != IDX_OK) wrong("trim failed");
    if (g_held != g_mem[(char *)kept].bytes) wrong("memory is held after the trim");
    put(kept, SB);
    void *p = get(6 * MiB, SA);
    use(p, SA);
    put(p, SA);
    g_no_wait = true;
    if (idx::cached_trim() == IDX_OK) wrong("trim without the device's synchronisation");
    g_no_wait = false;
    if (get(6 * MiB, SA) != p) wrong("the block was lost");
}

// A block of device 0 freed with device 1 current: its null stream is another.
void other_device() {
    void *p = get(3 * MiB, S0);
    g_dev = 1;
    (void)hipDeviceSynchronize();
    use(p, S0);
    put(p, S0);
    g_dev = 0;
    if (!get(3 * MiB, S0)) wrong("no memory");
}

// What the null stream left idle does not push out another stream's blocks.
void null_left_idle() {
    std::vector<void *> p;
    for (int i = 0; i < 8; ++i) p.push_back(get((900 + 30 * i) * MiB, S0));
    for (void *q : p) put(q, S0);
    void *mine = get(3000 * MiB, SA);
    for (int i = 0; i < 5; ++i) {
        put(mine, SA);
        if (get(3000 * MiB, SA) != mine) return wrong("a stream's own block was not kept");
    }
}

struct Scenario { const char *name; void (*run)(); };
const Scenario kAll[] = {{"order", order}, {"capture_elsewhere", capture_elsewhere},
                         {"failed_wait", failed_wait}, {"memory_short", memory_short},
                         {"trim", trim}, {"other_device", other_device},
                         {"null_left_idle", null_left_idle}};

}  // namespace

int main(int argc, char **argv) {
    for (const Scenario &s : kAll)
        if (argc == 2 && !strcmp(argv[1], s.name)) {
            s.run();
            for (const std::string &w : g_wrong) printf("%s\n", w.c_str());
            return g_wrong.empty() ? 0 : 1;
        }
    printf("no such scenario\n");
    return 2;
}
