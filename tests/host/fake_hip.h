// A HIP runtime for host tests of libqaoa.so: the executable defines the runtime
// calls that the library makes, so they resolve here and no GPU is touched.  Device
// memory is host memory filled with a pattern, copies are memcpy, and kernel
// launches are logged by name; the few kernels that a test needs the effect of are
// carried out on the host (run_kernel).
#pragma once
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

struct Fake {
    std::map<const void *, std::string> kernels;  // host stub -> device name
    std::vector<std::string> log;                 // launches and pinned allocations, in order
    std::map<void *, size_t> live;                // device allocations
    size_t free_bytes = 1ull << 40;               // reported as free
    size_t largest = ~(size_t)0;                  // allocations above this fail
    size_t budget = ~(size_t)0, taken = 0;        // bytes to be had and live
    hipError_t last_error = hipSuccess;           // of a failed call, until it is read
    bool pin_fails = false;
    int pins = 0, mallocs = 0, copies = 0, streams = 0;
    char *pinned = nullptr;                       // memory that a caller has pinned
    size_t pinned_bytes = 0;
    std::map<void *, int> owner;                  // allocations of other devices than 0
    dim3 grid, block;                             // of the launch being pushed
    size_t shared = 0;
    hipStream_t stream = nullptr;
    std::string last;                             // name of the last launched kernel
};
inline Fake &fake()
{
    static Fake *f = new Fake;  // registrations come before main's statics
    return *f;
}

inline int launches(const char *part)
{
    int c = 0;
    for (const std::string &s : fake().log) c += s.find(part) != std::string::npos;
    return c;
}

#define EXPECT(cond)                                                     \
    do {                                                                 \
        if (!(cond)) {                                                   \
            std::printf("%s:%d: %s\n", __FILE__, __LINE__, #cond);       \
            std::exit(1);                                                \
        }                                                                \
    } while (0)

// The effect of the kernels that move entries (arguments as the kernels take them).
struct Entry16 {
    uint64_t a, b;
};
template <typename W>
inline void host_unfold(void **a)
{
    const W *in = *(const W **)a[0];
    const uint64_t half = *(uint64_t *)a[1];
    const uint32_t words = *(uint32_t *)a[2];
    W *out = *(W **)a[3];
    for (uint64_t i = 0; i < half * words; ++i) {
        out[i] = in[i];
        out[(2 * half - 1 - i / words) * words + i % words] = in[i];
    }
}
template <typename W>
inline void host_reverse(void **a)
{
    W *x = *(W **)a[0];
    std::reverse(x, x + *(uint64_t *)a[1]);
}
inline void run_kernel(const std::string &name, void **args)
{
    const bool w16 = name.find("HIP_vector_type") != std::string::npos, w8 = name.find("Im") != std::string::npos;
    if (name.find("k_reverse") != std::string::npos) w16 ? host_reverse<Entry16>(args) : host_reverse<uint64_t>(args);
    if (name.find("k_unfold_words") != std::string::npos) w16 ? host_unfold<Entry16>(args) : w8 ? host_unfold<uint64_t>(args) : host_unfold<uint32_t>(args);
    if (name.find("k_scan_final") != std::string::npos) **(double **)args[5] = 1.0;  // the total
    if (name.find("k_unfold_widen") != std::string::npos) {
        const float *in = *(const float **)args[0];
        const uint64_t half = *(uint64_t *)args[1];
        double *out = *(double **)args[2];
        for (uint64_t z = 0; z < half; ++z) out[z] = out[2 * half - 1 - z] = (double)in[z];
    }
}

extern "C" {

void **__hipRegisterFatBinary(const void *)
{
    static void *h;
    return &h;
}
void __hipRegisterFunction(void **, const void *stub, char *, const char *name, unsigned, void *, void *, void *, void *, int *)
{
    fake().kernels[stub] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t st)
{
    fake().grid = g;
    fake().block = b;
    fake().shared = s;
    fake().stream = st;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *s, hipStream_t *st)
{
    *g = fake().grid;
    *b = fake().block;
    *s = fake().shared;
    *st = fake().stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **args, size_t, hipStream_t)
{
    fake().last = fake().kernels[f];
    fake().log.push_back(fake().last);
    run_kernel(fake().last, args);
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t bytes)
{
    ++fake().mallocs;
    *p = nullptr;
    if (bytes > fake().largest || bytes > fake().budget - fake().taken) return fake().last_error = hipErrorOutOfMemory;
    uint8_t *q = (uint8_t *)std::malloc(bytes);
    for (size_t i = 0; i < bytes; ++i) q[i] = (uint8_t)(i * 37 + (i >> 8) * 11 + (i >> 16) * 5 + 1) & 0x3f;
    fake().live[q] = bytes;
    fake().taken += bytes;
    *p = q;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    if (!p) return hipSuccess;
    const auto it = fake().live.find(p);
    EXPECT(it != fake().live.end());
    fake().taken -= it->second;
    fake().live.erase(it);
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned)
{
    ++fake().pins;
    fake().log.push_back("pin");
    *p = fake().pin_fails ? nullptr : std::calloc(bytes, 1);
    return *p ? hipSuccess : fake().last_error = hipErrorOutOfMemory;
}
hipError_t hipHostFree(void *p)
{
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemGetInfo(size_t *fr, size_t *tot)
{
    *fr = fake().free_bytes;
    *tot = 1ull << 40;
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    ++fake().copies;
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t)
{
    std::memset(d, v, n);
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p)
{
    std::memset(a, 0, sizeof *a);
    const char *c = (const char *)p;
    if (c >= fake().pinned && c < fake().pinned + fake().pinned_bytes) {
        a->type = hipMemoryTypeHost;
        a->hostPointer = a->devicePointer = (void *)p;
        return hipSuccess;
    }
    const auto it = fake().live.upper_bound((void *)p);
    if (it == fake().live.begin() || c >= (const char *)std::prev(it)->first + std::prev(it)->second) return hipErrorInvalidValue;
    a->type = hipMemoryTypeDevice;
    const auto of = fake().owner.find(std::prev(it)->first);
    a->device = of == fake().owner.end() ? 0 : of->second;
    a->devicePointer = (void *)p;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int)
{
    *v = 100000;
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int)
{
    std::memset((void *)p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t)
{
    *n = 2;
    return hipSuccess;
}
hipError_t hipGetLastError(void)
{
    const hipError_t e = fake().last_error;
    fake().last_error = hipSuccess;
    return e;
}
const char *hipGetErrorString(hipError_t) { return "fake"; }
hipError_t hipGetSymbolAddress(void **, const void *) { return hipErrorInvalidValue; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned)
{
    ++fake().streams;
    *s = (hipStream_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s)
{
    std::free((void *)s);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g)
{
    *g = nullptr;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t)
{
    *e = (hipGraphExec_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t e)
{
    std::free((void *)e);
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned)
{
    *e = (hipEvent_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e)
{
    std::free((void *)e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t)
{
    fake().log.push_back("event");
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t)
{
    *ms = 0.f;
    return hipSuccess;
}

}  // extern "C"
