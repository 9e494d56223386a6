// Large copies from device to the caller's pageable memory.
//
// The runtime's own copy to pageable memory reaches 18 GB/s here, a third of
// the link, and the caller's fresh pages are faulted in by its one thread.
// Instead the data comes through a ring of pinned buffers at the link's rate
// (57 GB/s) and a few threads move it on, which also shares the page faults.
// Drawing and reading 92 MB of walks: 15.5 -> 9.5 ms; packing a corpus and
// reading its 88 MB: 10.8 -> 7.0 ms.
//
// The rings belong to the process: one copy takes a ring of its own, at most
// kRingsKept (16 MB each) wait for the next copy, and the last context to be
// destroyed frees them.
#include <algorithm>
#include <atomic>
#include <cstring>
#include <exception>
#include <mutex>
#include <new>
#include <thread>
#include <utility>

#include "common.h"

namespace felog {

namespace {

constexpr size_t kSlotBytes = (size_t)2 << 20;
constexpr int kSlots = 8;
constexpr int kRingsKept = 2;
constexpr int kCopyThreads = 4;                        // the calling one among them
constexpr size_t kStagedMin = (size_t)4 << 20;         // smaller copies go directly
constexpr size_t kThreadsMin = (size_t)16 << 20;       // smaller ones stay on one thread

struct Ring {
    int device = -1;
    char* buf = nullptr;
    hipEvent_t ev[kSlots] = {};
    ~Ring()
    {
        for (hipEvent_t e : ev)
            if (e) (void)hipEventDestroy(e);
        if (buf) (void)hipHostFree(buf);
    }
};

std::mutex g_mu;
Ring* g_rings[kRingsKept] = {};   // waiting for a copy; no destructor at exit
int g_contexts = 0;

// A ring on the device, or none when pinned memory or events are short.
std::unique_ptr<Ring> take_ring(int device)
{
    {
        std::lock_guard<std::mutex> lk(g_mu);
        for (Ring*& w : g_rings)
            if (w && w->device == device) return std::unique_ptr<Ring>(std::exchange(w, nullptr));
    }
    std::unique_ptr<Ring> r(new (std::nothrow) Ring);
    if (!r) return nullptr;
    r->device = device;
    void* p = nullptr;
    // another thread's capture is not disturbed by the allocation
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    bool ok = hipHostMalloc(&p, kSlots * kSlotBytes, hipHostMallocDefault) == hipSuccess;
    r->buf = static_cast<char*>(p);
    for (hipEvent_t& e : r->ev)
        ok = ok && hipEventCreateWithFlags(&e, hipEventDisableTiming) == hipSuccess;
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    if (!ok) {
        (void)hipGetLastError();
        return nullptr;
    }
    return r;
}

void give_ring(std::unique_ptr<Ring> r)
{
    std::lock_guard<std::mutex> lk(g_mu);
    if (g_contexts == 0) return;
    for (Ring*& w : g_rings)
        if (!w) {
            w = r.release();
            return;
        }
}

// True for memory the device copies to directly (pinned by the caller).
bool pinned(const void* p)
{
    hipPointerAttribute_t a{};
    if (hipPointerGetAttributes(&a, p) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return a.type != hipMemoryTypeUnregistered;
}

struct Copy {
    char* dst;
    size_t bytes;
    int64_t chunks;
    Ring& ring;
    std::atomic<int64_t> issued{0}, next{0};
    std::atomic<int64_t> done[kSlots] = {};   // chunks that have left the slot
    std::atomic<int> error{0};                // hipError_t, or -1 to stop

    size_t size_of(int64_t c) const
    {
        return std::min(kSlotBytes, bytes - (size_t)c * kSlotBytes);
    }
    // Moves chunk c, whose copy has been issued, to the caller's memory.
    void move(int64_t c)
    {
        const int slot = (int)(c % kSlots);
        const hipError_t e = hipEventSynchronize(ring.ev[slot]);
        if (e != hipSuccess) error.store((int)e);
        else
            std::memcpy(dst + (size_t)c * kSlotBytes, ring.buf + slot * kSlotBytes, size_of(c));
        done[slot].store(c / kSlots + 1, std::memory_order_release);
    }
    void work()
    {
        for (;;) {
            const int64_t c = next.fetch_add(1);
            if (c >= chunks) return;
            while (issued.load(std::memory_order_acquire) <= c) {
                if (error.load()) return;
                std::this_thread::yield();
            }
            move(c);
        }
    }
};

}  // namespace

void host_copies_attach()
{
    std::lock_guard<std::mutex> lk(g_mu);
    ++g_contexts;
}

void host_copies_detach()
{
    std::lock_guard<std::mutex> lk(g_mu);
    if (--g_contexts > 0) return;
    for (Ring*& w : g_rings) delete std::exchange(w, nullptr);
}

void copy_to_host(const Ctx& c, void* dst, const void* src, size_t bytes)
{
    c.make_current();   // a ring's events are of the device that is current when it is made
    std::unique_ptr<Ring> ring;
    if (bytes >= kStagedMin && !pinned(dst)) ring = take_ring(c.device);
    if (!ring) {
        FELOG_HIP(hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, c.stream));
        c.sync();
        return;
    }
    c.sync();   // the threads wait for copies only, not for the work before them
    Copy cp{static_cast<char*>(dst), bytes, (int64_t)((bytes + kSlotBytes - 1) / kSlotBytes), *ring};
    std::thread threads[kCopyThreads - 1];
    bool alone = true;
    if (bytes >= kThreadsMin) {
        try {
            for (std::thread& t : threads) {
                t = std::thread([&cp, dev = c.device] {
                    (void)hipSetDevice(dev);
                    cp.work();
                });
                alone = false;
            }
        } catch (const std::exception&) {
            // fewer threads
        }
    }
    hipError_t err = hipSuccess;
    for (int64_t k = 0; k < cp.chunks && err == hipSuccess && !cp.error.load(); ++k) {
        const int slot = (int)(k % kSlots);
        // the slot's previous chunk must have left it
        while (cp.done[slot].load(std::memory_order_acquire) < k / kSlots && !cp.error.load()) {
            if (alone) cp.move(cp.next.fetch_add(1));
            else std::this_thread::yield();
        }
        err = hipMemcpyAsync(ring->buf + slot * kSlotBytes,
                             static_cast<const char*>(src) + (size_t)k * kSlotBytes, cp.size_of(k),
                             hipMemcpyDeviceToHost, c.stream);
        if (err == hipSuccess) err = hipEventRecord(ring->ev[slot], c.stream);
        if (err == hipSuccess) cp.issued.store(k + 1, std::memory_order_release);
    }
    if (err != hipSuccess) cp.error.store(-1);
    cp.work();
    for (std::thread& t : threads)
        if (t.joinable()) t.join();
    const hipError_t se = hipStreamSynchronize(c.stream);   // nothing writes the ring any more
    if (err == hipSuccess && cp.error.load() > 0) err = (hipError_t)cp.error.load();
    if (err == hipSuccess) err = se;
    FELOG_HIP(err);
    give_ring(std::move(ring));
}

}  // namespace felog
