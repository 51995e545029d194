// The part of the HIP runtime the library calls, on the CPU and without a device:
// allocations are host memory, copies are copies, kernels are only named.  Linked
// into a host-only build of the library, it shows which calls allocate, wait and
// launch what, and lets a call fail, with no GPU.  Every call appends a line to a log:
//   malloc BYTES | free | hostmalloc BYTES | hostfree | sync | launch KERNEL GX GY GZ
//   bad CALL (a pointer or event that is not, or no longer, the library's)
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>

namespace {

std::string g_log;
std::map<const void*, std::string>& kernels() {     // filled while the library is being loaded
    static std::map<const void*, std::string> m;
    return m;
}
std::map<void*, size_t> g_host;          // live pinned allocations
std::set<void*> g_device, g_events;      // live device allocations and events
long long g_fail_host_from = -1;         // pinned allocations of at least this many bytes fail
long long g_fail_malloc_from = -1;       // device allocations of at least this many bytes fail
std::string g_fail_call;                 // the next call of this name fails
bool g_pending = false;                  // events are not complete when asked
unsigned long long g_totals[3] = {0, 0, 0};
hipError_t g_last = hipSuccess;          // as the runtime keeps it: a failed call's error, until it is asked for

void note(const char* what, long long n = -1) {
    g_log += what;
    if (n >= 0) g_log += " " + std::to_string(n);
    g_log += "\n";
}

bool fails(const char* call) {
    if (g_fail_call != call) return false;
    g_fail_call.clear();
    return true;
}

struct Config {
    dim3 grid, block;
    size_t shared;
    hipStream_t stream;
} g_config;

int g_handle;                            // any non-null object
template <class T>
T handle() { return reinterpret_cast<T>(&g_handle); }

}  // namespace

extern "C" {

const char* fake_log() { return g_log.c_str(); }
void fake_clear() { g_log.clear(); }
void fake_fail_host_from(long long bytes) { g_fail_host_from = bytes; }
void fake_fail_malloc_from(long long bytes) { g_fail_malloc_from = bytes; }
void fake_fail_call(const char* name) { g_fail_call = name; }
void fake_pending(int on) { g_pending = on != 0; }
unsigned long long fake_host_bytes() {
    unsigned long long n = 0;
    for (const auto& h : g_host) n += h.second;
    return n;
}
// what a replayed graph leaves in every pinned allocation of three 64-bit words (the
// coded bits, 0xFF bytes and pinned bytes of a JPEG stream)
void fake_graph_totals(unsigned long long a, unsigned long long b, unsigned long long c) {
    g_totals[0] = a, g_totals[1] = b, g_totals[2] = c;
}

hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { note("sync"); return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
    std::memset(p, 0, sizeof *p);
    std::strcpy(p->gcnArchName, "gfx950");
    p->multiProcessorCount = 256;
    p->warpSize = 64;
    return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "fake error"; }
hipError_t hipGetLastError() {
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}

hipError_t hipMalloc(void** p, size_t n) {
    note("malloc", (long long)n);
    if (fails("hipMalloc") || (g_fail_malloc_from >= 0 && (long long)n >= g_fail_malloc_from))
        return g_last = hipErrorOutOfMemory;
    *p = std::calloc(1, n);
    if (!*p) return g_last = hipErrorOutOfMemory;
    g_device.insert(*p);
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    if (!p) return hipSuccess;
    note("free");
    if (!g_device.erase(p)) {
        note("bad hipFree");
        return g_last = hipErrorInvalidValue;
    }
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    note("hostmalloc", (long long)n);
    if (fails("hipHostMalloc") || (g_fail_host_from >= 0 && (long long)n >= g_fail_host_from))
        return g_last = hipErrorOutOfMemory;
    *p = std::calloc(1, n);
    g_host[*p] = n;
    return hipSuccess;
}
hipError_t hipHostFree(void* p) {
    if (p) note("hostfree");
    g_host.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemset(void* p, int v, size_t n) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(d, s, n);
    return hipSuccess;
}

hipError_t hipStreamCreate(hipStream_t* s) { *s = handle<hipStream_t>(); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    if (fails("hipStreamCreateWithFlags")) return g_last = hipErrorOutOfMemory;
    *s = handle<hipStream_t>();
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { note("sync"); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { *g = handle<hipGraph_t>(); return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
    *e = handle<hipGraphExec_t>();
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) {
    note("graph");
    if (fails("hipGraphLaunch")) return g_last = hipErrorUnknown;
    for (auto& h : g_host)
        if (h.second == sizeof g_totals) std::memcpy(h.first, g_totals, sizeof g_totals);
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
    if (fails("hipEventCreate")) return g_last = hipErrorOutOfMemory;
    *e = reinterpret_cast<hipEvent_t>(std::malloc(1));
    g_events.insert(*e);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) {
    if (!g_events.erase(e)) {
        note("bad hipEventDestroy");
        return g_last = hipErrorInvalidHandle;
    }
    std::free(e);
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t) { return g_pending ? hipErrorNotReady : hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
    if (!g_events.count(e)) note("bad hipEventRecord");
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
    static char scratch[64];
    *p = scratch;
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 4; return hipSuccess; }

hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream) {
    g_config = {grid, block, shared, stream};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* stream) {
    *grid = g_config.grid, *block = g_config.block, *shared = g_config.shared, *stream = g_config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void**, size_t, hipStream_t) {
    g_log += "launch " + kernels()[f] + " " + std::to_string(grid.x) + " " + std::to_string(grid.y) + " " +
             std::to_string(grid.z) + "\n";
    if (fails("hipLaunchKernel")) g_last = hipErrorLaunchFailure;
    return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) {
    static void* module;
    return &module;
}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    kernels()[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}

}  // extern "C"
