// Device memory that outlives a call: the kept workspaces of evaluation calls.
#include <mutex>
#include <new>

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

}  // namespace

// Give back the device's kept workspaces whose calls are over (the current device).
void spaces_drop(int dev)
{
    OutsideCapture guard;
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
        if (e != hipSuccess) {
            (void)hipGetLastError();
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
