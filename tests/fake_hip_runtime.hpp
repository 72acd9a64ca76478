// A HIP runtime without a device, for tests of the host code: memory is never touched, kernels are recorded by name and not run, and a test decides
// which allocations fail, how long a kernel takes and whether a launch throws.
#pragma once
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <new>
#include <string>
#include <vector>

namespace fake {

std::map<void*, size_t> live;                                    // allocations
std::vector<size_t> asked;                                       // sizes asked for
std::vector<std::string> launched;                               // kernel names, mangled
std::function<bool(size_t)> refuse = [](size_t) { return false; };
std::function<float(const std::string&)> takes = [](const std::string&) { return 1.f; };      // ms between two events, from the last kernel launched
bool launch_throws = false;

std::map<const void*, std::string>& kernels() { static std::map<const void*, std::string> k; return k; }      // filled before main

struct Launch { dim3 grid, block; size_t shared; hipStream_t stream; };
std::vector<Launch> pushed;
char scratch[16];

bool ran(const char* part)
{
    for (const auto& k : launched)
        if (k.find(part) != std::string::npos) return true;
    return false;
}

}  // namespace fake

extern "C" {

hipError_t hipMalloc(void** p, size_t bytes)
{
    fake::asked.push_back(bytes);
    if (fake::refuse(bytes)) { *p = nullptr; return hipErrorOutOfMemory; }
    *p = std::aligned_alloc(256, 256);                           // an address of its own; what lies there is never read
    fake::live[*p] = bytes;
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    if (!p) return hipSuccess;
    if (!fake::live.erase(p)) std::abort();                      // freed twice, or never allocated
    std::free(p);
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void**, size_t, hipStream_t)
{
    if (fake::launch_throws) throw std::bad_alloc();
    fake::launched.push_back(fake::kernels()[f]);
    return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t)
{
    *ms = fake::takes(fake::launched.empty() ? std::string() : fake::launched.back());
    return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { fake::kernels()[host] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t s)
{
    fake::pushed.push_back({grid, block, shared, s});
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* s)
{
    const fake::Launch l = fake::pushed.back();
    fake::pushed.pop_back();
    *grid = l.grid; *block = l.block; *shared = l.shared; *s = l.stream;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = reinterpret_cast<hipEvent_t>(&fake::scratch); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) { std::memset(p, 0, sizeof *p); p->multiProcessorCount = 256; return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "fake error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { *p = fake::scratch; return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphGetNodes(hipGraph_t, hipGraphNode_t*, size_t* n) { *n = 0; return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipMemset(void*, int, size_t) { return hipSuccess; }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 2; return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }

}  // extern "C"
