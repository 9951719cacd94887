// The library's memory functions (csrc/memory.cpp) on a runtime of this file's own: device
// memory of a given size, streams whose work ends when the test says so.
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <mutex>
#include <set>
#include <thread>
#include <vector>

#include "pndf_internal.h"

namespace {
std::mutex mu;
std::map<void*, size_t> live;                 // device memory
std::atomic<size_t> room{1000}, in_use{0};
std::map<hipStream_t, long> issued, ended;    // work on a stream: counts of issued and ended calls
struct Event { hipStream_t s = nullptr; long at = 0; };
std::set<void*> events;
std::atomic<int> mallocs{0}, frees{0}, async_mallocs{0}, async_frees{0}, waits{0}, syncs{0};
thread_local bool capturing = false;
std::atomic<bool> sync_blocks{false};

hipError_t get(void** p, size_t bytes)
{
    std::lock_guard<std::mutex> l(mu);
    if (in_use + bytes > room) return hipErrorOutOfMemory;
    *p = std::malloc(16);
    live[*p] = bytes;
    in_use += bytes;
    return hipSuccess;
}
hipError_t put(void* p)
{
    std::lock_guard<std::mutex> l(mu);
    auto it = live.find(p);
    if (it == live.end()) { std::printf("freed twice or unknown\n"); std::exit(3); }
    in_use -= it->second;
    live.erase(it);
    return hipSuccess;
}
}  // namespace

extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { ++mallocs; return get(p, n); }
hipError_t hipFree(void* p) { ++frees; return put(p); }
hipError_t hipMallocAsync(void** p, size_t n, hipStream_t) { ++async_mallocs; return get(p, n); }
hipError_t hipFreeAsync(void* p, hipStream_t) { ++async_frees; return put(p); }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { Event* x = new Event; std::lock_guard<std::mutex> l(mu); events.insert(x); *e = (hipEvent_t)x; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { std::lock_guard<std::mutex> l(mu); events.erase((void*)e); delete (Event*)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { std::lock_guard<std::mutex> l(mu); *(Event*)e = Event{s, issued[s]}; return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t e) { std::lock_guard<std::mutex> l(mu); Event* x = (Event*)e; return ended[x->s] >= x->at ? hipSuccess : hipErrorNotReady; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { ++waits; return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* c) { *c = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t* d) { *d = (size_t)s >= 1000 ? 1 : 0; return hipSuccess; }
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode*) { return hipSuccess; }
hipError_t hipDeviceSynchronize(void)
{
    ++syncs;
    while (sync_blocks) std::this_thread::sleep_for(std::chrono::milliseconds(1));
    std::lock_guard<std::mutex> l(mu);
    for (auto& s : issued) ended[s.first] = s.second;
    return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* a, size_t* t) { *a = room - in_use; *t = room; return hipSuccess; }
}

#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); std::exit(1); } } while (0)

static void work(hipStream_t s) { std::lock_guard<std::mutex> l(mu); ++issued[s]; }
static void end(hipStream_t s) { std::lock_guard<std::mutex> l(mu); ended[s] = issued[s]; }

int main()
{
    using namespace pndf;
    const hipStream_t A = (hipStream_t)1, B = (hipStream_t)2, other = (hipStream_t)1000;
    const size_t MB = (size_t)1 << 20;
    void *p, *q, *r;
    // ---- workspaces: the same stream has a space again at once, another when it is over
    room = 4096 * MB;
    CHECK(stream_alloc(&p, MB, A) == hipSuccess); work(A); stream_free(p, A);
    CHECK(stream_alloc(&q, MB - 4000, A) == hipSuccess && q == p && waits == 1);
    work(A); stream_free(q, A);
    CHECK(stream_alloc(&q, MB, B) == hipSuccess && q != p);
    work(B); stream_free(q, B); end(A); end(B);
    CHECK(stream_alloc(&r, MB, B) == hipSuccess && (r == p || r == q)); stream_free(r, B);
    CHECK(async_mallocs == 2 && async_frees == 0);
    // the smallest that holds it
    CHECK(stream_alloc(&r, 64 * MB, A) == hipSuccess); stream_free(r, A);
    CHECK(stream_alloc(&q, MB, A) == hipSuccess && q != r); stream_free(q, A);
    // two at once on one stream are two
    CHECK(stream_alloc(&p, MB, A) == hipSuccess && stream_alloc(&q, MB, A) == hipSuccess && p != q);
    stream_free(p, A); stream_free(q, A);
    // bounded; what is over makes room, what is not stays
    for (int k = 0; k < 12; ++k) { CHECK(stream_alloc(&p, (100 + 20 * k) * MB, A) == hipSuccess); stream_free(p, A); }
    CHECK(in_use <= kStreamKeep);
    CHECK(stream_alloc(&p, 400 * MB, A) == hipSuccess && stream_alloc(&q, 400 * MB, B) == hipSuccess);
    work(A); work(B); stream_free(p, A); stream_free(q, B);
    CHECK(in_use <= kStreamKeep);
    CHECK(stream_alloc(&p, 1000 * MB, A) == hipSuccess); stream_free(p, A);
    CHECK(in_use <= kStreamKeep);
    // under capture and on another device's stream the runtime's own calls
    capturing = true;
    int n = async_frees;
    CHECK(stream_alloc(&p, MB, A) == hipSuccess); stream_free(p, A);
    CHECK(async_frees == n + 1);
    capturing = false;
    CHECK(stream_alloc(&p, MB, other) == hipSuccess); stream_free(p, other);
    CHECK(async_frees == n + 2);
    // ---- blocks: kept for the next handle of about the size; a smaller one has its own
    CHECK(block_alloc(10 * MB, &p) == hipSuccess && block_alloc(30 * MB, &q) == hipSuccess);
    block_free(p);
    CHECK(in_use >= 40 * MB);
    n = mallocs;
    CHECK(block_alloc(9 * MB + MB / 2, &r) == hipSuccess && r == p && mallocs == n);
    block_free(r);
    CHECK(block_alloc(5 * MB, &r) == hipSuccess && r != p && mallocs == n + 1);
    block_free(r);
    // at most 1 / 128 of the device: larger ones go at once, the oldest make room
    CHECK(block_alloc(33 * MB, &r) == hipSuccess); n = frees; block_free(r); CHECK(frees == n + 1);
    CHECK(block_alloc(28 * MB, &r) == hipSuccess); block_free(r);
    CHECK(frees == n + 3);   // 10 and 5
    // ---- with the last handle the workspaces go, after a while the blocks
    work(A); end(A);
    CHECK(in_use > 58 * MB);
    block_free(q);
    CHECK(in_use == 30 * MB);
    for (int k = 0; k < 300 && in_use; ++k) std::this_thread::sleep_for(std::chrono::milliseconds(10));
    CHECK(in_use == 0 && events.empty());
    // (and again: the thread had ended)
    CHECK(block_alloc(10 * MB, &p) == hipSuccess); block_free(p);
    for (int k = 0; k < 300 && in_use; ++k) std::this_thread::sleep_for(std::chrono::milliseconds(10));
    CHECK(in_use == 0);
    // ---- no memory: whatever asks has what is kept
    for (int kind = 0; kind < 3; ++kind) {
        room = 4096 * MB;
        CHECK(block_alloc(MB, &q) == hipSuccess);   // (a handle)
        CHECK(block_alloc(20 * MB, &p) == hipSuccess); block_free(p);
        CHECK(stream_alloc(&p, 300 * MB, A) == hipSuccess); work(A); stream_free(p, A);
        room = in_use + 10 * MB;
        const size_t ask = 200 * MB;
        if (kind == 0) { CHECK(device_alloc(&r, 320 * MB) == hipSuccess); (void)hipFree(r); }
        if (kind == 1) { CHECK(block_alloc(320 * MB, &r) == hipSuccess); block_free(r); }
        if (kind == 2) { CHECK(stream_alloc(&r, 320 * MB, B) == hipSuccess); stream_free(r, B); }
        CHECK(device_alloc(&r, ask * 10) == hipErrorOutOfMemory);
        CHECK(block_alloc(ask * 10, &r) == hipErrorOutOfMemory && stream_alloc(&r, ask * 10, A) == hipErrorOutOfMemory);
        block_free(q);
        for (int k = 0; k < 300 && in_use; ++k) std::this_thread::sleep_for(std::chrono::milliseconds(10));
        CHECK(in_use == 0);
    }
    // ---- a release that waits for the device holds nobody up
    room = 4096 * MB;
    CHECK(block_alloc(MB, &p) == hipSuccess && block_alloc(2 * MB, &q) == hipSuccess);
    sync_blocks = true;
    n = syncs;
    std::thread t([&] { block_free(p); });
    while (syncs == n) std::this_thread::yield();
    std::atomic<bool> got{false};
    std::thread u([&] { void* x; got = block_alloc(3 * MB, &x) == hipSuccess; });
    for (int k = 0; k < 300 && !got; ++k) std::this_thread::sleep_for(std::chrono::milliseconds(10));
    CHECK(got);
    sync_blocks = false;
    t.join();
    u.join();
    // ---- threads: what two hold at once is never the same
    std::vector<std::thread> ts;
    std::set<void*> held;
    std::mutex hm;
    std::atomic<bool> bad{false};
    for (int k = 0; k < 4; ++k)
        ts.emplace_back([&, k] {
            for (int i = 0; i < 300; ++i) {
                void *x, *y;
                const hipStream_t s = (hipStream_t)(size_t)(10 + (k + i) % 3);
                if (stream_alloc(&x, (1 + i % 5) * MB, s) != hipSuccess || block_alloc((1 + i % 3) * MB, &y) != hipSuccess) { bad = true; return; }
                {
                    std::lock_guard<std::mutex> l(hm);
                    bad = bad || !held.insert(x).second || !held.insert(y).second;
                }
                work(s);
                {
                    std::lock_guard<std::mutex> l(hm);
                    held.erase(x);
                    held.erase(y);
                }
                stream_free(x, s);
                block_free(y);
            }
        });
    for (auto& x : ts) x.join();
    CHECK(!bad);
    std::printf("ok\n");
    return 0;
}
