// Device memory behind the default allocator: a bounded cache of freed blocks.
//
// Builds, merges, training and range calls take and free buffers of up to a
// few GiB each.  The runtime's pool returned a build's freed blocks to the
// driver when the next block was freed, also with its release threshold raised
// (ROCm 7.2, thresholds of 2^36 to 2^64 - 1 bytes), so every build unmapped and
// mapped its temporaries again: about 0.6 ms per build of 2^26 64-bit keys, and
// 20 to 40 ms once the driver had handed out all the memory it had cleared
// beforehand.  Blocks freed here stay mapped and serve the next request of
// about their size.
//
// Rules:
//   * A block carries an event recorded on the stream that freed it; the
//     stream that takes it next waits for that event, so any stream and any
//     thread may take it.  A block that the null stream freed has none (a
//     record and a wait cost a range call 21 us of 2555 on its two scratch
//     blocks): calls on the null stream alone take it again or give it back.
//     A call on another stream does no work on the null stream, which would
//     break a capture that any thread has under way.
//   * At most kCacheBytes and kCacheBlocks idle blocks are kept per device, of
//     those that a call reaches (twice that in all, where the null stream's are
//     not used again while other streams work); a block not taken again within
//     kCacheAge requests is given back to the runtime's pool, and all idle
//     blocks are, through it, to the driver when an allocation of any size
//     fails, or on request (cached_trim).
//   * A stream under graph capture bypasses the cache: its allocations and
//     frees become graph nodes, as without it.
#include <mutex>
#include <new>
#include <unordered_map>
#include <vector>

#include "internal.hpp"

namespace idx {
namespace {

constexpr size_t kCacheBytes = 8ull << 30;  // the temporaries of a 2^27-lookup or 2^26-key call, several times over
constexpr size_t kCacheBlocks = 256;
constexpr uint64_t kCacheAge = 256;         // requests an idle block outlives

struct Block {
    void *p;
    size_t bytes;
    int dev;
    hipEvent_t ev;   // recorded where the block was last freed, unless on_null
    bool on_null;    // last freed on the null stream, whose calls alone may touch it
    uint64_t tick;   // request count at that time
};

struct Cache {
    std::mutex mu;
    std::vector<Block> idle;                  // oldest first
    std::unordered_map<void *, Block> taken;  // blocks handed out
    uint64_t tick = 0;
};

// Never destroyed: handles may be closed while the process ends.
Cache *cache() {
    static Cache *c = new (std::nothrow) Cache();
    return c;
}

// Requests are rounded to 1/64 of their size, so repeated calls of about the
// same size meet the same blocks.
size_t rounded(size_t bytes) {
    size_t step = 4096;
    while (step * 128 <= bytes) step <<= 1;
    return (bytes + step - 1) / step * step;
}

// Orders `s` after the work that used b (b.dev is the current device); false:
// neither the stream nor the host can wait for it, and b stays as it is.
bool wait_for(const Block &b, hipStream_t s) {
    if (b.on_null) return true;  // s is the null stream
    if (hipStreamWaitEvent(s, b.ev, 0) == hipSuccess || hipEventSynchronize(b.ev) == hipSuccess) return true;
    (void)hipGetLastError();
    return false;
}

// Back to the idle blocks, the next to be evicted (without host memory for
// that, b is lost).
void restore(Cache *c, const Block &b) {
    try {
        std::lock_guard<std::mutex> lock(c->mu);
        c->taken.erase(b.p);
        c->idle.insert(c->idle.begin(), b);
    } catch (...) {
    }
}

// Blocks back to the driver, after the work that used them.
void give_back(Cache *c, const std::vector<Block> &gone, hipStream_t s) {
    for (const Block &b : gone) {
        if (!wait_for(b, s)) {
            restore(c, b);
            continue;
        }
        (void)hipFreeAsync(b.p, s);
        (void)hipEventDestroy(b.ev);
    }
    (void)hipGetLastError();
}

// Whether a call on stream s of device dev may take b or give it back.
bool reach(const Block &b, int dev, hipStream_t s) { return b.dev == dev && (!b.on_null || s == nullptr); }

// Moves the idle blocks beyond the bounds (all: every one), of those that a call
// on stream s of device dev reaches, from the cache to `gone`.
void evict(Cache *c, int dev, hipStream_t s, bool all, std::vector<Block> &gone) {
    size_t bytes = 0, blocks = 0;
    for (size_t i = c->idle.size(); i-- > 0;) {  // newest first
        const Block &b = c->idle[i];
        if (!reach(b, dev, s)) continue;
        bytes += b.bytes;
        ++blocks;
        if (all || bytes > kCacheBytes || blocks > kCacheBlocks || c->tick - b.tick > kCacheAge) {
            gone.push_back(b);
            bytes -= b.bytes;
            --blocks;
            c->idle.erase(c->idle.begin() + (long)i);
        }
    }
}

// Raises the release threshold of the runtime's pool, so that what the cache
// gives back, and blocks too large for it, need not go to the driver at the
// next synchronisation (which the first graph replay over a new batch of 338
// handles met: 620 against 340 us).  How much of it the pool then keeps is the
// runtime's choice; trim_pool empties it.
void keep_pool() {
    static thread_local int done_dev = -1;
    int dev = 0;
    if (hipGetDevice(&dev) == hipSuccess && dev != done_dev) {
        hipMemPool_t pool;
        if (hipDeviceGetDefaultMemPool(&pool, dev) == hipSuccess) {
            uint64_t thr = ~0ull;
            (void)hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &thr);
        }
        done_dev = dev;
    }
    (void)hipGetLastError();
}

void *plain_get(size_t bytes, hipStream_t s, hipError_t *err) {
    keep_pool();
    void *p = nullptr;
    *err = hipMallocAsync(&p, bytes, s);
    if (*err == hipSuccess) return p;
    (void)hipGetLastError();
    return nullptr;
}

// Device dev's idle blocks that a call on s reaches, to the runtime's pool.
void give_back_idle(Cache *c, int dev, hipStream_t s) {
    std::vector<Block> gone;
    try {
        std::lock_guard<std::mutex> lock(c->mu);
        evict(c, dev, s, true, gone);
    } catch (...) {  // host memory: what was found so far
    }
    give_back(c, gone, s);
    (void)hipStreamSynchronize(s);
    (void)hipGetLastError();
}

// What the runtime's pool keeps, to the driver.
void trim_pool(int dev) {
    hipMemPool_t pool;
    if (hipDeviceGetDefaultMemPool(&pool, dev) == hipSuccess) (void)hipMemPoolTrimTo(pool, 0);
    (void)hipGetLastError();
}

// Device dev's idle blocks back to the driver, with what the runtime's pool
// keeps: for a call on s that found no memory.  The null stream's blocks go
// too, unless a capture is under way that work on the null stream would break.
void give_back_all(Cache *c, int dev, hipStream_t s) {
    give_back_idle(c, dev, s);
    if (s != nullptr && !capturing(nullptr)) give_back_idle(c, dev, nullptr);
    trim_pool(dev);
}

}  // namespace

bool capturing(hipStream_t s) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) != hipSuccess) {
        (void)hipGetLastError();
        return true;
    }
    return st != hipStreamCaptureStatusNone;
}

void *cached_get(size_t bytes, hipStream_t s, hipError_t *err) {
    Cache *c = cache();
    int dev = 0;
    if (!c || hipGetDevice(&dev) != hipSuccess || capturing(s)) {
        (void)hipGetLastError();
        return plain_get(bytes, s, err);
    }
    if (bytes > kCacheBytes) {  // not kept when it is freed
        void *p = plain_get(bytes, s, err);
        if (p) return p;
        give_back_all(c, dev, s);
        return plain_get(bytes, s, err);
    }
    const size_t want = rounded(bytes);
    std::vector<Block> gone;
    Block b{nullptr, want, dev, nullptr, false, 0};
    try {
        std::lock_guard<std::mutex> lock(c->mu);
        ++c->tick;
        size_t best = c->idle.size();
        for (size_t i = 0; i < c->idle.size(); ++i) {
            const Block &f = c->idle[i];
            if (reach(f, dev, s) && f.bytes >= want && f.bytes <= want + want / 4 &&
                (best == c->idle.size() || f.bytes <= c->idle[best].bytes))
                best = i;
        }
        if (best < c->idle.size()) {
            c->taken.emplace(c->idle[best].p, c->idle[best]);  // may throw: nothing is taken then
            b = c->idle[best];
            c->idle.erase(c->idle.begin() + (long)best);
        }
        evict(c, dev, s, false, gone);
    } catch (...) {  // host memory: what was found so far stands
    }
    give_back(c, gone, s);
    gone.clear();
    *err = hipSuccess;
    if (b.p) {
        if (wait_for(b, s)) return b.p;
        restore(c, b);
        b = Block{nullptr, want, dev, nullptr, false, 0};
    }
    b.p = plain_get(want, s, err);
    if (!b.p) {
        give_back_all(c, dev, s);
        return plain_get(bytes, s, err);
    }
    if (hipEventCreateWithFlags(&b.ev, hipEventDisableTiming) != hipSuccess) {
        (void)hipGetLastError();
        return b.p;  // not registered: freed directly
    }
    try {
        std::lock_guard<std::mutex> lock(c->mu);
        c->taken.emplace(b.p, b);
    } catch (...) {
        (void)hipEventDestroy(b.ev);
    }
    return b.p;
}

int cached_trim() {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return hip_fail(e);
    }
    if (Cache *c = cache()) give_back_idle(c, dev, nullptr);
    trim_pool(dev);
    return IDX_OK;
}

void cached_put(void *p, hipStream_t s) {
    Cache *c = cache();
    std::vector<Block> gone;
    bool kept = false;
    if (c) {
        std::lock_guard<std::mutex> lock(c->mu);
        const auto it = c->taken.find(p);
        if (it != c->taken.end()) {
            Block b = it->second;
            c->taken.erase(it);
            try {
                int dev = -1;  // s may belong to another device than the block: not kept then
                b.on_null = s == nullptr;
                if (hipGetDevice(&dev) == hipSuccess && dev == b.dev && !capturing(s) &&
                    (b.on_null || hipEventRecord(b.ev, s) == hipSuccess)) {
                    b.tick = c->tick;
                    c->idle.push_back(b);
                    kept = true;
                    evict(c, b.dev, s, false, gone);
                }
            } catch (...) {  // host memory
            }
            if (!kept) {
                (void)hipGetLastError();
                (void)hipEventDestroy(b.ev);
            }
        }
    }
    if (!kept) (void)hipFreeAsync(p, s);
    give_back(c, gone, s);
}

}  // namespace idx
