// A HIP runtime for tests on the CPU that runs no kernel: device memory is
// host memory, copies are made at once, and every call that queues or waits
// is written to a log, one line each.  Loaded (global) before the library, it
// takes the place of the runtime the library links.
//
//   HIP_RECORDER_LOG   the log file
//   HIP_RECORDER_FAIL  calls that fail, comma-separated: a kernel's name (or
//                      part of it), "*" for every kernel, or #k, the k-th
//                      logged call that may fail (from 0)
//
// Lines: "copy S dst bytes", "launch S name grid block", "record E S",
// "wait S E", "sync S", "alloc kind bytes", "device-sync", "event-sync E".
// Streams and events are numbered from 1; a line of a failed call ends in
// " failed".  A launch of 2^32 or more threads fails, as on a device.
#define __HIP_PLATFORM_AMD__ 1
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
std::map<const void *, std::string> &names()
{
    static auto *m = new std::map<const void *, std::string>;
    return *m;
}

FILE *out()
{
    static FILE *f = fopen(getenv("HIP_RECORDER_LOG"), "w");
    return f;
}

bool fails(const char *kernel)
{
    static long k = 0;
    const char *e = getenv("HIP_RECORDER_FAIL");
    const std::string want = std::string(",") + (e ? e : "") + ",", nth = ",#" + std::to_string(k++) + ",";
    if (want.find(nth) != std::string::npos) return true;
    for (size_t a = 1; kernel && a < want.size();) {
        const size_t b = want.find(',', a);
        const std::string w = want.substr(a, b - a);
        if (w == "*" || (!w.empty() && std::string(kernel).find(w) != std::string::npos)) return true;
        a = b + 1;
    }
    return false;
}

template <class... A>
hipError_t note(hipError_t err, const char *fmt, A... a)
{
    if constexpr (sizeof...(a) != 0) fprintf(out(), fmt, a...);
    else fputs(fmt, out());
    fprintf(out(), "%s\n", err == hipSuccess ? "" : " failed");
    fflush(out());
    return err;
}

long counter = 0;
struct Handle {
    long id;
};
long id(const void *h) { return h ? ((const Handle *)h)->id : 0; }

hipError_t last = hipSuccess;  // (one thread launches at a time here)
hipError_t launch(const char *name, dim3 g, dim3 b, hipStream_t s)
{
    const unsigned long long n = 1ull * g.x * b.x;
    hipError_t e = g.x == 0 || n >> 32 ? hipErrorInvalidConfiguration : hipSuccess;
    if (fails(name)) e = hipErrorLaunchFailure;
    return last = note(e, "launch %ld %s %u %u", id(s), name, g.x, b.x);
}
dim3 pushed[2];
size_t pushed_shm;
hipStream_t pushed_stream;
}  // namespace

extern "C" {

void **__hipRegisterFatBinary(const void *)
{
    static void *h;
    return &h;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *,
                           void *, int *)
{
    names()[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t shm, hipStream_t s)
{
    pushed[0] = g;
    pushed[1] = b;
    pushed_shm = shm;
    pushed_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *shm, hipStream_t *s)
{
    *g = pushed[0];
    *b = pushed[1];
    *shm = pushed_shm;
    *s = pushed_stream;
    return hipSuccess;
}

hipError_t hipGetDevice(int *d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int)
{
    memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int)
{
    *v = 100000;
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t e) { return e == hipSuccess ? "no error" : "recorded error"; }
hipError_t hipGetLastError()
{
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}

hipError_t hipMalloc(void **p, size_t n)
{
    if (n >> 30) return note(hipErrorOutOfMemory, "alloc device %zu", n);
    *p = aligned_alloc(256, (n + 255) / 256 * 256);
    return note(hipSuccess, "alloc device %zu", n);
}
hipError_t hipFree(void *p)
{
    free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    *p = aligned_alloc(256, (n + 255) / 256 * 256);
    return note(hipSuccess, "alloc host %zu", n);
}
hipError_t hipHostFree(void *p)
{
    free(p);
    return hipSuccess;
}
hipError_t hipMallocAsync(void **p, size_t n, hipStream_t)
{
    *p = aligned_alloc(256, (n + 255) / 256 * 256);
    return note(hipSuccess, "alloc async %zu", n);
}
hipError_t hipFreeAsync(void *p, hipStream_t)
{
    free(p);
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *)
{
    static void *a = aligned_alloc(256, 8 << 20);
    *p = a;
    return hipSuccess;
}

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned)
{
    *s = (hipStream_t) new Handle{++counter};
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *c)
{
    *c = hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned)
{
    *e = (hipEvent_t) new Handle{++counter};
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t)
{
    *ms = 1.0f;
    return hipSuccess;
}

hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st)
{
    const hipError_t e = fails(nullptr) ? hipErrorUnknown : hipSuccess;
    if (e == hipSuccess) memcpy(d, s, n);
    return note(e, "copy %ld %p %zu", id(st), d, n);
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t)
{
    memset(d, v, n);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t st)
{
    return note(fails(nullptr) ? hipErrorUnknown : hipSuccess, "record %ld %ld", id(e), id(st));
}
hipError_t hipStreamWaitEvent(hipStream_t st, hipEvent_t e, unsigned)
{
    return note(fails(nullptr) ? hipErrorUnknown : hipSuccess, "wait %ld %ld", id(st), id(e));
}
hipError_t hipStreamSynchronize(hipStream_t st) { return note(hipSuccess, "sync %ld", id(st)); }
hipError_t hipDeviceSynchronize() { return note(hipSuccess, "device-sync"); }
hipError_t hipEventSynchronize(hipEvent_t e) { return note(hipSuccess, "event-sync %ld", id(e)); }

hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **, size_t, hipStream_t st)
{
    return launch(names()[f].c_str(), g, b, st);
}
hipError_t hipModuleLoadData(hipModule_t *m, const void *)
{
    *m = (hipModule_t) new Handle{++counter};
    return hipSuccess;
}
hipError_t hipModuleUnload(hipModule_t) { return hipSuccess; }
hipError_t hipModuleGetFunction(hipFunction_t *f, hipModule_t, const char *name)
{
    *f = (hipFunction_t)strdup(name);
    return hipSuccess;
}
hipError_t hipModuleLaunchKernel(hipFunction_t f, unsigned gx, unsigned, unsigned, unsigned bx, unsigned, unsigned,
                                 unsigned, hipStream_t st, void **, void **)
{
    return launch((const char *)f, dim3(gx), dim3(bx), st);
}

}  // extern "C"
