// host_copy.hip -- large copies from device to pageable host memory.
//
// Handed to the runtime, such a copy runs through its staging buffer with one
// host thread, which also takes the page faults of a fresh destination: about
// 11 GB/s, and reading both fields of the 512^3 electrode (1.08 GB) took 98 ms
// beside the 160 ms of 100 fused steps. Here the device writes 4 MiB pieces
// into pinned memory while a few threads move the finished ones to the
// destination.
//
// The pinned area (32 MiB, one per process) is made by the first large copy
// and freed with the last solver. A copy that finds it taken by another
// thread, or that cannot have it or its threads, goes to the runtime.
#include "host_copy_internal.h"

#include <algorithm>
#include <atomic>
#include <cstring>
#include <mutex>
#include <thread>

namespace cdi {

namespace {

constexpr uint64_t kPiece = 4ull << 20;
constexpr int kSlots = 8, kThreads = 8;

std::mutex g_mu;
void *g_area = nullptr;
bool g_taken = false;
int g_users = 0;

// Pinned memory is made and freed whatever is captured meanwhile, in this thread
// or another: it takes no part in a graph, and the default mode would have the
// call refused and the capture invalidated.
struct WhileCapturing {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    WhileCapturing() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~WhileCapturing() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

void free_area()
{
    WhileCapturing relaxed;
    (void)hipHostFree(g_area);
    g_area = nullptr;
}

void *take_area()
{
    std::lock_guard<std::mutex> lock(g_mu);
    if (g_taken) return nullptr;
    WhileCapturing relaxed;
    if (!g_area && hipHostMalloc(&g_area, kPiece * kSlots, hipHostMallocPortable) != hipSuccess) {
        (void)hipGetLastError();
        g_area = nullptr;
        return nullptr;
    }
    g_taken = true;
    return g_area;
}

void give_area()
{
    std::lock_guard<std::mutex> lock(g_mu);
    g_taken = false;
    if (g_users <= 0) free_area();
}

hipError_t plain_copy(void *dst, const void *src, uint64_t bytes, hipStream_t s)
{
    const hipError_t e = hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, s);
    return e != hipSuccess ? e : hipStreamSynchronize(s);
}

// Slot q of the area serves pieces q, q + kSlots, ...: worker q waits for the
// piece's event, moves it out and sends the slot's next piece on its way.
hipError_t staged_copy(uint8_t *area, uint8_t *dst, const uint8_t *src, uint64_t bytes, hipStream_t s)
{
    int dev = 0;  // the stream's: the caller's current device may be another
    hipError_t err = s ? hipStreamGetDevice(s, &dev) : hipGetDevice(&dev);
    if (err != hipSuccess) return err;
    const int64_t pieces = (int64_t)((bytes + kPiece - 1) / kPiece);
    std::atomic<int> failed{hipSuccess};
    auto size = [&](int64_t k) { return std::min<uint64_t>(kPiece, bytes - (uint64_t)k * kPiece); };
    auto serve = [&](int q) {
        hipError_t e = hipSetDevice(dev);
        hipEvent_t ev = nullptr;
        if (e == hipSuccess) e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
        uint8_t *slot = area + (uint64_t)q * kPiece;
        auto send = [&](int64_t k) {
            hipError_t r = hipMemcpyAsync(slot, src + (uint64_t)k * kPiece, size(k), hipMemcpyDeviceToHost, s);
            return r != hipSuccess ? r : hipEventRecord(ev, s);
        };
        if (e == hipSuccess && q < pieces) e = send(q);
        for (int64_t k = q; e == hipSuccess && k < pieces; k += kSlots) {
            e = hipEventSynchronize(ev);
            if (e != hipSuccess) break;
            std::memcpy(dst + (uint64_t)k * kPiece, slot, size(k));
            if (k + kSlots < pieces) e = send(k + kSlots);
        }
        if (ev) {
            if (e != hipSuccess) (void)hipStreamSynchronize(s);  // nothing may still write the slot
            (void)hipEventDestroy(ev);
        }
        if (e != hipSuccess) failed = e;
    };
    static_assert(kThreads == kSlots, "a worker per slot");
    std::thread workers[kThreads];
    int started = 0;
    try {
        for (; started < kThreads - 1; ++started) workers[started] = std::thread(serve, started);
    } catch (...) {  // no more threads: this one serves the rest
    }
    for (int q = started; q < kThreads; ++q) serve(q);
    for (int q = 0; q < started; ++q) workers[q].join();
    return (hipError_t)failed.load();
}

}  // namespace

hipError_t copy_to_host(void *dst, const void *src, uint64_t bytes, hipStream_t s)
{
    // (hipStreamPerThread names another stream in every worker)
    void *area = bytes >= kStagedCopyMin && s != hipStreamPerThread ? take_area() : nullptr;
    if (!area) return plain_copy(dst, src, bytes, s);
    const hipError_t e = staged_copy((uint8_t *)area, (uint8_t *)dst, (const uint8_t *)src, bytes, s);
    give_area();
    return e;
}

void staging_user_added()
{
    std::lock_guard<std::mutex> lock(g_mu);
    ++g_users;
}

void staging_user_removed()
{
    std::lock_guard<std::mutex> lock(g_mu);
    if (--g_users <= 0 && !g_taken && g_area) free_area();
}

}  // namespace cdi
