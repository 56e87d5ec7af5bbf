// A HIP runtime without a device, for tests of the library's host code on a machine that has no GPU: linked with the
// library's objects (tests/stub_library.py) in place of libamdhip64.  "Device" memory is host memory, a launch runs nothing
// and notes the kernel's name, grid, workgroup and LDS bytes, and an allocation larger than a limit fails as the real one
// does when the device is full.  The stub_* functions set and read this from the test.
#include <hip/hip_runtime_api.h>

#include <cxxabi.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>

namespace {

struct Call {
    dim3 grid, block;
    size_t lds = 0;
    hipStream_t stream = nullptr;
} pending;

// (made on first use: the objects register their kernels from constructors of their own)
std::map<const void*, std::string>& kernels()
{
    static std::map<const void*, std::string> m;
    return m;
}
std::map<void*, size_t> device_memory;
std::map<std::pair<int, const void*>, size_t> lds_limit;     // per device: what a kernel's dynamic LDS was raised to
int device = 0;
std::string launched;                       // one line per launch: name grid.x grid.y grid.z block lds
size_t limit = ~(size_t)0, allocated = 0, freed = 0, peak = 0;      // peak: largest allocation since it was reset
int units = 256;
size_t taken = 0;                           // device memory that others hold
bool capturing = false;
std::string failing;                        // launches of kernels with this name fail
hipError_t last_error = hipSuccess;
int event_word, stream_word;

} // namespace

extern "C" {

void stub_reset()
{
    launched.clear();
    limit = ~(size_t)0;
    allocated = freed = 0;
    capturing = false;
    failing.clear();
}
void stub_fail(const char* kernel) { failing = kernel; }
const char* stub_launches() { return launched.c_str(); }
void stub_units(int n) { units = n; }
void stub_taken(size_t bytes) { taken = bytes; }
void stub_limit(size_t bytes) { limit = bytes; }
void stub_capturing(int on) { capturing = on != 0; }
size_t stub_allocated() { return allocated; }
size_t stub_freed() { return freed; }
size_t stub_peak() { return peak; }
void stub_peak_reset() { peak = 0; }

void** __hipRegisterFatBinary(const void*)
{
    static void* handle = nullptr;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, dim3*, dim3*, int*)
{
    int status = 0;
    char* plain = abi::__cxa_demangle(name, nullptr, nullptr, &status);
    std::string s = plain ? plain : name;
    free(plain);
    const size_t paren = s.find('(');
    if (paren != std::string::npos) s.resize(paren);
    if (s.rfind("void ", 0) == 0) s.erase(0, 5);
    if (s.rfind("som::", 0) == 0) s.erase(0, 5);
    for (size_t at; (at = s.find(' ')) != std::string::npos;) s.erase(at, 1);
    kernels()[host] = s;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream)
{
    pending.grid = grid;
    pending.block = block;
    pending.lds = lds;
    pending.stream = stream;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream)
{
    *grid = pending.grid;
    *block = pending.block;
    *lds = pending.lds;
    *stream = pending.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void**, size_t lds, hipStream_t)
{
    const auto it = kernels().find(f);
    if (!failing.empty() && it != kernels().end() && it->second.rfind(failing, 0) == 0) return last_error = hipErrorLaunchFailure;
    const auto raised = lds_limit.find({device, f});
    if (lds > (raised == lds_limit.end() ? 64 * 1024 : raised->second)) return last_error = hipErrorInvalidValue;
    char sizes[128];
    snprintf(sizes, sizeof(sizes), " %u %u %u %u %zu\n", grid.x, grid.y, grid.z, block.x, lds);
    launched += (it == kernels().end() ? std::string("?") : it->second) + sizes;
    return grid.x && grid.y && grid.z && block.x ? hipSuccess : hipErrorInvalidConfiguration;
}

hipError_t hipMalloc(void** p, size_t bytes)
{
    if (bytes > limit) return hipErrorOutOfMemory;
    *p = malloc(bytes ? bytes : 1);
    device_memory[*p] = bytes;
    allocated += bytes;
    if (bytes > peak) peak = bytes;
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    const auto it = device_memory.find(p);
    if (it == device_memory.end()) return hipErrorInvalidValue;
    freed += it->second;
    device_memory.erase(it);
    free(p);
    return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* left, size_t* total)
{
    *total = (size_t)288 << 30;
    *left = *total - taken - (allocated - freed);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) { return hipMalloc(p, bytes); }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipMemset(void* p, int v, size_t bytes)
{
    memset(p, v, bytes);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* to, const void* from, size_t bytes, hipMemcpyKind, hipStream_t)
{
    memcpy(to, from, bytes);
    return hipSuccess;
}
hipError_t hipMemcpy(void* to, const void* from, size_t bytes, hipMemcpyKind)
{
    memcpy(to, from, bytes);
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* at, const void*)
{
    memset(at, 0, sizeof(*at));
    at->type = hipMemoryTypeDevice;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*)
{
    static double none[1];
    *p = none;
    return hipSuccess;
}

hipError_t hipGetDeviceCount(int* n)
{
    *n = 2;
    return hipSuccess;
}
hipError_t hipSetDevice(int d)
{
    device = d;
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* prop, int)
{
    memset(prop, 0, sizeof(*prop));
    strcpy(prop->gcnArchName, "gfx950:sramecc+:xnack-");
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t which, int)
{
    *v = which == hipDeviceAttributeMultiprocessorCount ? units : 256;
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute, int bytes)
{
    lds_limit[{device, f}] = (size_t)bytes;
    return hipSuccess;
}
hipError_t hipGetLastError()
{
    const hipError_t e = last_error;
    last_error = hipSuccess;
    return e;
}
const char* hipGetErrorString(hipError_t) { return "an error of the stub"; }

hipError_t hipEventCreate(hipEvent_t* e)
{
    *e = (hipEvent_t)&event_word;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t)
{
    *ms = 0.0f;
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned)
{
    *s = (hipStream_t)&stream_word;
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* status)
{
    *status = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}

} // extern "C"

// what a program that was linked with this stub gave back, on its way out
__attribute__((destructor)) static void stub_report()
{
    if (getenv("STUB_REPORT")) fprintf(stderr, "stub: %zu bytes allocated, %zu freed\n", allocated, freed);
}
