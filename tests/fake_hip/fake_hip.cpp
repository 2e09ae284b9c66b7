// A stand-in for the HIP runtime, preloaded by the CPU tests of the library's host code: memory is host memory, launches are
// written down instead of run, and the test decides what the runtime answers.  One thread at a time.
#include <hip/hip_runtime_api.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <new>
#include <string>
#include <vector>

namespace {

struct Launch {
    std::string name;  // mangled
    unsigned grid[3], block[3];
    size_t smem;
    unsigned char arg1[64];  // the plan kernel's second argument, else zeros
};

std::map<const void *, std::string> &names() {
    static std::map<const void *, std::string> m;
    return m;
}
std::vector<Launch> launches;
hipError_t pending = hipSuccess;       // what hipGetLastError() has to say
hipError_t launch_error = hipSuccess;  // what a launch returns (nothing is enqueued then)
hipError_t sync_error = hipSuccess;    // what waiting for an event or the device returns
hipError_t copy_error = hipSuccess;    // what an asynchronous copy returns
hipError_t status_error = hipSuccess;  // what asking for a stream's capture status returns
bool capturing = false;
size_t largest_new = ~(size_t)0;  // a larger operator new throws
long event_waits = 0;

hipError_t fail(hipError_t e) {
    if (e != hipSuccess) pending = e;
    return e;
}

hipError_t record(const void *f, dim3 g, dim3 b, void **args, size_t smem) {
    if (launch_error != hipSuccess) return fail(launch_error);
    Launch l;
    l.name = names()[f];
    const unsigned gg[3] = {g.x, g.y, g.z}, bb[3] = {b.x, b.y, b.z};
    memcpy(l.grid, gg, sizeof gg);
    memcpy(l.block, bb, sizeof bb);
    l.smem = smem;
    memset(l.arg1, 0, sizeof l.arg1);
    if (l.name.find("plan_apply_kernel") != std::string::npos) memcpy(l.arg1, args[1], 24);
    launches.push_back(l);
    return hipSuccess;
}

struct Config {
    dim3 grid, block;
    size_t smem;
    hipStream_t stream;
};
Config config;

}  // namespace

void *operator new(size_t n) {
    void *p = n <= largest_new ? malloc(n ? n : 1) : nullptr;
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }

extern "C" {

// ---- what the tests steer and read ----
void fake_reset() {
    launches.clear();
    pending = launch_error = sync_error = copy_error = status_error = hipSuccess;
    capturing = false;
    event_waits = 0;
}
void fake_set(const char *what, int v) {
    if (!strcmp(what, "pending")) pending = (hipError_t)v;
    if (!strcmp(what, "launch_error")) launch_error = (hipError_t)v;
    if (!strcmp(what, "sync_error")) sync_error = (hipError_t)v;
    if (!strcmp(what, "copy_error")) copy_error = (hipError_t)v;
    if (!strcmp(what, "status_error")) status_error = (hipError_t)v;
    if (!strcmp(what, "largest_new")) largest_new = (size_t)v;
    if (!strcmp(what, "capturing")) capturing = v != 0;
}
int fake_launches() { return (int)launches.size(); }
const char *fake_name(int i) { return launches[i].name.c_str(); }
void fake_dims(int i, unsigned *out) {
    memcpy(out, launches[i].grid, 12);
    memcpy(out + 3, launches[i].block, 12);
}
const void *fake_arg1(int i) { return launches[i].arg1; }
long fake_event_waits() { return event_waits; }

// ---- registration ----
void **__hipRegisterFatBinary(const void *) {
    static void *handle = nullptr;
    return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *device_name, unsigned, void *, void *, dim3 *, dim3 *, int *) {
    names()[host] = device_name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}

// ---- launches ----
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t smem, hipStream_t s) {
    config = Config{g, b, smem, s};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *smem, hipStream_t *s) {
    *g = config.grid;
    *b = config.block;
    *smem = config.smem;
    *s = config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t smem, hipStream_t) { return record(f, g, b, args, smem); }
hipError_t hipExtLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t smem, hipStream_t, hipEvent_t, hipEvent_t, int) {
    return record(f, g, b, args, smem);
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }

// ---- errors, devices ----
hipError_t hipGetLastError() {
    const hipError_t e = pending;
    pending = hipSuccess;
    return e;
}
hipError_t hipGetDeviceCount(int *n) {
    *n = 1;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int d) { return d == 0 ? hipSuccess : fail(hipErrorInvalidDevice); }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
    memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    return hipSuccess;
}

// ---- memory ----
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    *p = aligned_alloc(256, (n + 255) & ~(size_t)255);
    return *p ? hipSuccess : fail(hipErrorOutOfMemory);
}
hipError_t hipHostFree(void *p) {
    free(p);
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) { return hipHostMalloc(p, n, 0); }
hipError_t hipFree(void *p) { return hipHostFree(p); }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind, hipStream_t) { return fail(copy_error); }  // (queued, never run)
hipError_t hipGetSymbolAddress(void **p, const void *) {
    *p = (void *)(uintptr_t)0x7f0000000000ull;  // (an address nothing else has; kernels do not run here)
    return hipSuccess;
}

// ---- streams, events ----
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) {
    *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return fail(status_error);
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return fail(sync_error); }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    *e = reinterpret_cast<hipEvent_t>(malloc(8));
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) {
    free(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) {
    ++event_waits;
    return fail(sync_error);
}
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
    *ms = 0.f;
    return hipSuccess;
}

}  // extern "C"
