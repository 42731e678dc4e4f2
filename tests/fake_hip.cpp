// A HIP runtime for host tests: preloaded before the library, it answers the
// calls of the library's host code without a GPU.  "Device" memory is host
// memory, copies copy, kernels do nothing, and every launch and fill is logged
// by kernel name, stream and whether that stream was capturing.  Failures
// are asked for through the fake_* calls.
#define __HIP_PLATFORM_AMD__ 1
#include <hip/hip_runtime_api.h>
#include <sys/mman.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

namespace {
std::mutex mu;
std::map<void *, size_t> maps;
std::map<const void *, std::string> names;
std::string events;
hipError_t last = hipSuccess;
size_t host_limit = ~size_t(0);
hipStream_t capturing = nullptr;
bool capture_on = false;

hipError_t done(hipError_t e)
{
    if (e != hipSuccess) last = e;
    return e;
}
bool captured(hipStream_t s) { return capture_on && s == capturing; }
void event(const std::string &what, hipStream_t s)
{
    std::lock_guard<std::mutex> lk(mu);
    events += what + (captured(s) ? " captured\n" : "\n");
}
void *take(size_t n)  // pages are backed only where touched
{
    n = n ? n : 16;
    void *p = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (p == MAP_FAILED) return nullptr;
    std::lock_guard<std::mutex> lk(mu);
    maps[p] = n;
    return p;
}
hipError_t give(void *p)
{
    if (!p) return hipSuccess;
    std::lock_guard<std::mutex> lk(mu);
    auto it = maps.find(p);
    if (it == maps.end()) return done(hipErrorInvalidValue);
    munmap(p, it->second);
    maps.erase(it);
    return hipSuccess;
}
}  // namespace

extern "C" {

// hipHostMalloc fails for more than this many bytes
void fake_host_limit(size_t bytes) { host_limit = bytes; }
void fake_capture(void *stream, int on) { capturing = (hipStream_t)stream, capture_on = on != 0; }
// the log since the last call
const char *fake_events()
{
    static std::string out;
    std::lock_guard<std::mutex> lk(mu);
    out.swap(events);
    events.clear();
    return out.c_str();
}

void **__hipRegisterFatBinary(const void *)
{
    static void *h;
    return &h;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, void *, void *, int *)
{
    names[f] = name;
}
static thread_local struct {
    dim3 grid, block;
    size_t shmem;
    hipStream_t s;
} conf;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t m, hipStream_t s)
{
    conf = {g, b, m, s};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *m, hipStream_t *s)
{
    *g = conf.grid, *b = conf.block, *m = conf.shmem, *s = conf.s;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **, size_t, hipStream_t s)
{
    event("launch " + names[f], s);
    return hipSuccess;
}

hipError_t hipGetDeviceCount(int *n) { return *n = 1, hipSuccess; }
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int)
{
    std::memset(p, 0, sizeof(*p));
    std::strcpy(p->gcnArchName, "gfx950:sramecc+:xnack-");
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipMemGetInfo(size_t *f, size_t *t) { return *f = *t = size_t(288) << 30, hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int threads, size_t)
{
    return *n = threads >= 1024 ? 1 : 1024 / threads, hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *)
{
    static void *q = take(size_t(64) << 20);
    return *p = q, hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) { return (*p = take(n)) ? hipSuccess : done(hipErrorOutOfMemory); }
hipError_t hipFree(void *p) { return give(p); }
hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    *p = n > host_limit ? nullptr : take(n);
    return *p ? hipSuccess : done(hipErrorOutOfMemory);
}
hipError_t hipHostFree(void *p) { return give(p); }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { return std::memcpy(d, s, n), hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st)
{
    event("copy", st);
    if (!captured(st)) std::memcpy(d, s, n);
    return hipSuccess;
}
// (not carried out: nothing reads device memory)
hipError_t hipMemset(void *, int, size_t) { return event("fill", nullptr), hipSuccess; }
hipError_t hipMemsetAsync(void *, int, size_t, hipStream_t s) { return event("fill", s), hipSuccess; }

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { return *s = (hipStream_t)std::malloc(8), hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { return std::free((void *)s), hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s)
{
    return captured(s) ? done(hipErrorStreamCaptureUnsupported) : hipSuccess;
}
hipError_t hipStreamQuery(hipStream_t s) { return hipStreamSynchronize(s); }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *c)
{
    return *c = captured(s) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone, hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return *e = (hipEvent_t)std::malloc(8), hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { return std::free((void *)e), hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = 1.f, hipSuccess; }
hipError_t hipGetLastError()
{
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
const char *hipGetErrorString(hipError_t) { return "fake HIP error"; }
}
