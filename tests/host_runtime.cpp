// A stand-in for the HIP runtime in tests of the library's host side without a GPU: memory is host memory, kernels are counted by
// name and not run (but for the copies out of pinned buffers, which are a memcpy), and a test says which launch fails.  Built as a shared object
// with the runtime's soname, so that the library under test loads it instead.
#include <hip/hip_runtime_api.h>

#include <atomic>
#include <chrono>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "host_runtime.h"

namespace {
std::mutex mutex;
std::map<const void *, std::string> names;   // kernels by the address of their host stub
std::vector<std::string> launched;           // in order; failed ones are not among them
std::string fail_name;
int fail_after = -1, fail_malloc_after = -1;
int64_t malloc_bytes = 0, copied_bytes = 0;
std::atomic<int> malloc_ms{0};
int event_records = 0;
thread_local hipError_t last_error = hipSuccess;
struct Call { dim3 grid, block; size_t lds; hipStream_t st; };
thread_local Call call;
}

extern "C" {

// ---- what tests use
void host_fail_launch(const char *kernel, int after) { std::lock_guard<std::mutex> l(mutex); fail_name = kernel; fail_after = after; }
void host_fail_malloc(int after) { std::lock_guard<std::mutex> l(mutex); fail_malloc_after = after; }
void host_set_last_error(int e) { last_error = (hipError_t)e; }
void host_malloc_takes(int ms) { malloc_ms = ms; }
int64_t host_malloc_bytes() { std::lock_guard<std::mutex> l(mutex); return malloc_bytes; }
int64_t host_copied_bytes() { std::lock_guard<std::mutex> l(mutex); return copied_bytes; }
int host_event_records() { std::lock_guard<std::mutex> l(mutex); return event_records; }
int host_launches(const char *kernel)
{
    std::lock_guard<std::mutex> l(mutex);
    int n = 0;
    for (const std::string &s : launched) n += s.find(kernel) != std::string::npos;
    return n;
}

// ---- the runtime
void **__hipRegisterFatBinary(const void *) { static void *module; return &module; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, dim3 *, dim3 *, int *)
{
    std::lock_guard<std::mutex> l(mutex);
    names[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t st) { call = {grid, block, lds, st}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *st)
{
    *grid = call.grid; *block = call.block; *lds = call.lds; *st = call.st;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **args, size_t, hipStream_t)
{
    std::lock_guard<std::mutex> l(mutex);
    const std::string &name = names[f];
    if (!fail_name.empty() && name.find(fail_name) != std::string::npos && fail_after-- == 0) return last_error = hipErrorLaunchFailure;
    launched.push_back(name);
    auto copy = [&](int first) {   // the arguments src, dst, pieces of 16 bytes
        const size_t bytes = *(size_t *)args[first + 2] * 16;
        if (bytes) std::memcpy(*(void **)args[first + 1], *(void **)args[first], bytes);
        copied_bytes += (int64_t)bytes;
    };
    if (name.find("copy_from_host") != std::string::npos) copy(0);
    if (name.find("pack_kv_tiles") != std::string::npos) copy(11);
    return hipSuccess;
}
hipError_t hipMalloc(void **out, size_t bytes)
{
    std::this_thread::sleep_for(std::chrono::milliseconds(malloc_ms));
    std::lock_guard<std::mutex> l(mutex);
    if (fail_malloc_after-- == 0) return last_error = hipErrorOutOfMemory;
    malloc_bytes += (int64_t)bytes;
    return (*out = std::malloc(bytes)) ? hipSuccess : (last_error = hipErrorOutOfMemory);
}
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **out, size_t bytes, unsigned) { return (*out = std::malloc(bytes)) ? hipSuccess : (last_error = hipErrorOutOfMemory); }
hipError_t hipMemcpy(void *to, const void *from, size_t n, hipMemcpyKind) { std::memcpy(to, from, n); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = (hipEvent_t)std::malloc(1); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { std::free((void *)e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { std::lock_guard<std::mutex> l(mutex); ++event_records; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { static char scratch[1]; *p = scratch; return hipSuccess; }
hipError_t hipGetLastError() { const hipError_t e = last_error; last_error = hipSuccess; return e; }
hipError_t hipPeekAtLastError() { return last_error; }
const char *hipGetErrorString(hipError_t) { return "an error"; }
}
