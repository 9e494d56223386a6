// copy_to_host on a runtime of two pretend devices, one of which is current: the
// HIP calls that it makes are defined here, with memory on the host and every
// copy done at once.  A stream belongs to the device of its number, an event and
// a pinned buffer to the device that was current when they were made, and, as
// in the runtime, an event is only recorded on a stream of its own device.
#include "hostcopy.cpp"

#include <cstdarg>
#include <cstdlib>

namespace felog {
void set_error(const char*, ...) {}
void clear_error() {}
void fail(felog_status code, const char* fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vfprintf(stderr, fmt, ap);
    va_end(ap);
    fputc('\n', stderr);
    throw Error{code};
}
void Ctx::make_current() const { (void)hipSetDevice(device); }
void Ctx::sync() const { FELOG_HIP(hipStreamSynchronize(stream)); }
DevBuf& DevBuf::operator=(DevBuf&&) noexcept { return *this; }
void DevBuf::release() {}
Model::~Model() {}
}  // namespace felog

static thread_local int t_device = 0;
static std::atomic<int> g_rings_made{0}, g_rings_freed{0};

struct Event {
    int device;
};
static int device_of(hipStream_t s) { return (int)(reinterpret_cast<intptr_t>(s) & 1); }

extern "C" {
hipError_t hipSetDevice(int d)
{
    t_device = d;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "refused"; }
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode*) { return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void*)
{
    a->type = hipMemoryTypeUnregistered;
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned)
{
    ++g_rings_made;
    *p = std::malloc(n);
    return hipSuccess;
}
hipError_t hipHostFree(void* p)
{
    ++g_rings_freed;
    std::free(p);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned)
{
    *e = reinterpret_cast<hipEvent_t>(new Event{t_device});
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e)
{
    delete reinterpret_cast<Event*>(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    return reinterpret_cast<Event*>(e)->device == device_of(s) ? hipSuccess
                                                                : hipErrorInvalidHandle;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t)
{
    std::memcpy(d, s, n);
    return hipSuccess;
}
}

int main()
{
    using namespace felog;
    Ctx c[2];
    for (int d = 0; d < 2; ++d) {
        c[d].device = d;
        c[d].stream = reinterpret_cast<hipStream_t>((intptr_t)(2 + d));
        host_copies_attach();
    }
    for (size_t bytes : {(size_t)4096, kStagedMin, kStagedMin + 1, kThreadsMin - 1, kThreadsMin,
                         (size_t)kSlots * kSlotBytes + 12345}) {
        std::vector<char> src(bytes), dst(bytes);
        for (size_t i = 0; i < bytes; ++i) src[i] = (char)(i * 2654435761u >> 13);
        for (int turn = 0; turn < 3; ++turn)
            for (int d = 0; d < 2; ++d) {   // device 0 is current before each
                (void)hipSetDevice(0);
                std::fill(dst.begin(), dst.end(), 0);
                try {
                    copy_to_host(c[d], dst.data(), src.data(), bytes);
                } catch (const Error&) {
                    fprintf(stderr, "%zu bytes from device %d failed\n", bytes, d);
                    return 1;
                }
                if (dst != src) {
                    fprintf(stderr, "%zu bytes from device %d differ\n", bytes, d);
                    return 1;
                }
            }
    }
    if (g_rings_made != 2) return 2;   // one per device, then kept
    for (int d = 0; d < 2; ++d) host_copies_detach();
    if (g_rings_freed != 2) return 3;
    puts("ok");
    return 0;
}
