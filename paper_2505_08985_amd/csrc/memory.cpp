// Device memory that outlives its user: the kept blocks of released handles and the kept
// workspaces of evaluation calls.  (No exception leaves these functions: lists are
// linked, their nodes allocated without throwing.)
#include <chrono>
#include <condition_variable>
#include <mutex>
#include <new>
#include <thread>

#include "pndf_internal.h"

namespace pndf {
namespace {

struct Space {
    void* p = nullptr;
    size_t size = 0;
    int dev = 0;
    hipStream_t stream = nullptr;  // of the call that had it last
    hipEvent_t done = nullptr;     // recorded there behind that call's work
    Space* next = nullptr;
};

struct Spaces {
    std::mutex mu;
    Space *kept = nullptr, *lent = nullptr;  // latest first
};

// (never destroyed: the runtime may be gone at exit)
Spaces& spaces()
{
    static Spaces* s = new Spaces;
    return *s;
}

// What the library does for itself is nobody's stream capture.
struct OutsideCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    OutsideCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~OutsideCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

bool over(hipEvent_t done)
{
    const hipError_t e = hipEventQuery(done);
    if (e != hipSuccess) (void)hipGetLastError();
    return e == hipSuccess;
}

// May a call on stream s have this space now?  Behind its last call if that was on the
// same stream, else once that call is over (streams never wait for each other).
bool ready(const Space& k, hipStream_t s)
{
    if (over(k.done)) return true;
    if (k.stream != s) return false;
    const hipError_t e = hipStreamWaitEvent(s, k.done, 0);
    if (e != hipSuccess) (void)hipGetLastError();
    return e == hipSuccess;
}

// Sizes in steps of an eighth to a quarter, so that calls of similar sizes share spaces.
size_t rounded(size_t bytes)
{
    size_t step = (size_t)1 << 16;
    while (step * 8 < bytes) step *= 2;
    return (bytes + step - 1) / step * step;
}

// Take the smallest kept space of `dev` that holds `bytes` and is ready; with the lock held.
Space* take(Spaces& w, int dev, size_t bytes, hipStream_t s)
{
    size_t above = bytes;  // sizes below were looked at
    const Space* last = nullptr;
    while (true) {
        Space** best = nullptr;
        for (Space** at = &w.kept; *at; at = &(*at)->next) {
            const Space* k = *at;
            if (k->dev != dev || k->size < above || (k->size == above && last && k <= last)) continue;
            if (!best || k->size < (*best)->size || (k->size == (*best)->size && k < *best)) best = at;
        }
        if (!best) return nullptr;
        Space* k = *best;
        if (ready(*k, s)) {
            *best = k->next;
            return k;
        }
        above = k->size;
        last = k;
    }
}

// Give back the device's kept workspaces whose calls are over (the current device).
void spaces_drop(int dev)
{
    Spaces& w = spaces();
    std::lock_guard<std::mutex> lock(w.mu);
    for (Space** at = &w.kept; *at;) {
        Space* k = *at;
        if (k->dev != dev || !over(k->done)) {
            at = &k->next;
            continue;
        }
        *at = k->next;
        (void)hipEventDestroy(k->done);
        (void)hipFree(k->p);
        delete k;
    }
}

using Clock = std::chrono::steady_clock;

struct Block {
    void* p = nullptr;
    size_t size = 0;
    int dev = 0;
    Clock::time_point since;
    Block* next = nullptr;
};

// Released blocks, latest first, and a thread that gives them back when their time is over;
// it exists while there are any.  (Never destroyed: handles may outlive the library's static
// objects.)
struct Blocks {
    std::mutex mu;
    std::condition_variable cv;
    Block *kept = nullptr, *used = nullptr;
    std::thread keeper;
    bool running = false, stop = false;
};

Blocks& blocks()
{
    static Blocks* b = new Blocks;
    return *b;
}

// Ends the thread at exit or when the library is unloaded.
struct KeeperEnd {
    ~KeeperEnd()
    {
        Blocks& b = blocks();
        {
            std::lock_guard<std::mutex> lock(b.mu);
            b.stop = true;
        }
        b.cv.notify_all();
        if (b.keeper.joinable()) b.keeper.join();
    }
};

void free_list(Block* b)
{
    OutsideCapture guard;
    int cur = -1;
    (void)hipGetDevice(&cur);
    while (b) {
        Block* const next = b->next;
        (void)hipSetDevice(b->dev);
        (void)hipFree(b->p);
        delete b;
        b = next;
    }
    if (cur >= 0) (void)hipSetDevice(cur);
}

// Unlink the kept blocks that match; with the lock held.
template <typename Pred>
Block* unlink(Blocks& b, Pred match)
{
    Block* out = nullptr;
    for (Block** at = &b.kept; *at;) {
        Block* const k = *at;
        if (!match(*k)) {
            at = &k->next;
            continue;
        }
        *at = k->next;
        k->next = out;
        out = k;
    }
    return out;
}

void keep_time(Blocks* b)
{
    const auto time = std::chrono::duration_cast<Clock::duration>(std::chrono::duration<double>(kBlockKeepSeconds));
    std::unique_lock<std::mutex> lock(b->mu);
    while (!b->stop && b->kept) {
        Clock::time_point first = b->kept->since;
        for (const Block* k = b->kept; k; k = k->next) first = k->since < first ? k->since : first;
        b->cv.wait_until(lock, first + time);
        const auto now = Clock::now();
        Block* const old = unlink(*b, [&](const Block& k) { return now - k.since >= time; });
        if (b->stop || !old) continue;  // (at exit what is unlinked goes with the process)
        lock.unlock();
        free_list(old);
        lock.lock();
    }
    b->running = false;
}

// Start the thread if there is none; with the lock held.  False if that fails.
bool keeper_runs(Blocks& b)
{
    static KeeperEnd end;  // (made after the runtime has started, so it goes before the runtime does)
    if (b.stop) return false;
    if (b.running) return true;
    try {
        if (b.keeper.joinable()) b.keeper.join();  // (it has left the lock for good)
        b.running = true;
        b.keeper = std::thread(keep_time, &b);
    } catch (...) {
        b.running = false;
    }
    return b.running;
}

// Give back everything that is kept on the current device.
void release_kept(int dev)
{
    OutsideCapture guard;
    if (hipDeviceSynchronize() == hipSuccess) spaces_drop(dev);
    (void)hipGetLastError();
    Blocks& b = blocks();
    Block* old;
    {
        std::lock_guard<std::mutex> lock(b.mu);
        old = unlink(b, [&](const Block& k) { return k.dev == dev; });
    }
    free_list(old);
}

}  // namespace

hipError_t device_alloc(void** p, size_t bytes)
{
    hipError_t e = hipMalloc(p, bytes);
    int dev = 0;
    if (e == hipErrorOutOfMemory && hipGetDevice(&dev) == hipSuccess) {
        (void)hipGetLastError();
        release_kept(dev);
        e = hipMalloc(p, bytes);
    }
    return e;
}

hipError_t block_alloc(size_t bytes, void** p)
{
    *p = nullptr;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    Blocks& b = blocks();
    Block* k = nullptr;
    {
        // the smallest kept block that holds it without wasting more than an eighth
        std::lock_guard<std::mutex> lock(b.mu);
        Block** best = nullptr;
        for (Block** at = &b.kept; *at; at = &(*at)->next) {
            const Block* o = *at;
            if (o->dev == dev && o->size >= bytes && o->size <= bytes + bytes / 8 && (!best || o->size < (*best)->size)) best = at;
        }
        if (best) {
            k = *best;
            *best = k->next;
        }
    }
    if (!k) {
        k = new (std::nothrow) Block;
        if (!k) return hipErrorOutOfMemory;
        k->dev = dev;
        k->size = bytes;
        e = device_alloc(&k->p, bytes);
        if (e != hipSuccess) {
            delete k;
            return e;
        }
    }
    *p = k->p;
    std::lock_guard<std::mutex> lock(b.mu);
    k->next = b.used;
    b.used = k;
    return hipSuccess;
}

void block_free(void* p)
{
    if (!p) return;
    Blocks& b = blocks();
    Block* k;
    bool last = true;
    {
        std::lock_guard<std::mutex> lock(b.mu);
        Block** at = &b.used;
        while (*at && (*at)->p != p) at = &(*at)->next;
        k = *at;
        if (!k) return;
        *at = k->next;
        for (const Block* o = b.used; o; o = o->next) last = last && o->dev != k->dev;
    }
    OutsideCapture guard;
    int cur = 0;
    size_t avail = 0, total = 0;
    bool keep = hipGetDevice(&cur) == hipSuccess && (cur == k->dev || hipSetDevice(k->dev) == hipSuccess);
    keep = keep && hipDeviceSynchronize() == hipSuccess;
    if (last && keep) spaces_drop(k->dev);
    keep = keep && hipMemGetInfo(&avail, &total) == hipSuccess && k->size <= total / kBlockKeepShare;
    (void)hipGetLastError();  // (a refused synchronisation is not the caller's error)
    k->next = nullptr;
    Block* old = k;
    if (keep) {
        std::lock_guard<std::mutex> lock(b.mu);
        k->since = Clock::now();
        k->next = b.kept;
        b.kept = k;
        // the oldest ones make room
        size_t held = 0;
        old = unlink(b, [&](const Block& o) {
            held += o.dev == k->dev ? o.size : 0;
            return o.dev == k->dev && held > total / kBlockKeepShare;
        });
        if (!keeper_runs(b)) {
            Block* mine = unlink(b, [](const Block&) { return true; });
            while (mine) {
                Block* const next = mine->next;
                mine->next = old;
                old = mine;
                mine = next;
            }
        }
    }
    free_list(old);
    (void)hipSetDevice(cur);
}

hipError_t stream_alloc(void** p, size_t bytes, hipStream_t s)
{
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    int dev = 0, cur = 0;
    const bool ours = hipStreamIsCapturing(s, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone &&
                      hipGetDevice(&cur) == hipSuccess && (!s || (hipStreamGetDevice(s, &dev) == hipSuccess && dev == cur));
    if (!ours) {
        (void)hipGetLastError();
        return hipMallocAsync(p, bytes, s);
    }
    OutsideCapture guard;
    Spaces& w = spaces();
    Space* k;
    {
        std::lock_guard<std::mutex> lock(w.mu);
        k = take(w, cur, bytes, s);
    }
    if (!k) {
        k = new (std::nothrow) Space;
        if (!k) return hipErrorOutOfMemory;
        k->dev = cur;
        k->size = rounded(bytes);
        hipError_t e = hipMallocAsync(&k->p, k->size, s);
        if (e == hipErrorOutOfMemory) {
            (void)hipGetLastError();
            release_kept(cur);
            k->size = bytes;
            e = hipMallocAsync(&k->p, bytes, s);
        }
        if (e == hipSuccess) {
            e = hipEventCreateWithFlags(&k->done, hipEventDisableTiming);
            if (e != hipSuccess) (void)hipFreeAsync(k->p, s);
        }
        if (e != hipSuccess) {
            delete k;
            return e;
        }
    }
    *p = k->p;
    std::lock_guard<std::mutex> lock(w.mu);
    k->next = w.lent;
    w.lent = k;
    return hipSuccess;
}

void stream_free(void* p, hipStream_t s)
{
    if (!p) return;
    Spaces& w = spaces();
    std::lock_guard<std::mutex> lock(w.mu);
    Space** at = &w.lent;
    while (*at && (*at)->p != p) at = &(*at)->next;
    Space* k = *at;
    if (!k) {
        (void)hipFreeAsync(p, s);
        return;
    }
    *at = k->next;
    OutsideCapture guard;
    // those that other calls have done with make room
    size_t held = k->size;
    for (const Space* o = w.kept; o; o = o->next) held += o->dev == k->dev ? o->size : 0;
    for (at = &w.kept; *at && held > kStreamKeep && k->size <= kStreamKeep;) {
        Space* o = *at;
        if (o->dev != k->dev || !ready(*o, s)) {
            at = &o->next;
            continue;
        }
        *at = o->next;
        held -= o->size;
        (void)hipEventDestroy(o->done);
        (void)hipFreeAsync(o->p, s);
        delete o;
    }
    k->stream = s;
    if (held <= kStreamKeep && hipEventRecord(k->done, s) == hipSuccess) {
        k->next = w.kept;
        w.kept = k;
        return;
    }
    (void)hipGetLastError();
    (void)hipEventDestroy(k->done);
    (void)hipFreeAsync(k->p, s);
    delete k;
}

}  // namespace pndf
