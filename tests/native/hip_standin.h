// A stand-in for the HIP runtime: the functions libfhp.so calls, over host
// memory, so that the library's host code runs without a GPU.  Kernels do not
// run; a test program sees every launch through on_launch and counts what the
// host does.  Included by exactly one source of a program, which links
// libfhp.so: the definitions here come before the runtime's.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>
#include <vector>

namespace standin {

struct Launch {
    std::string name;  // mangled
    uint32_t grid, block;
    void** args;
};

struct Counts {
    long launches, copies, waits, fills;
};

static std::map<const void*, std::string>& kernels() {
    static std::map<const void*, std::string> k;
    return k;
}
static Counts counts;
static std::string order;  // f fill, l other launch, c copy, w wait, in the order of their calls
static void (*on_launch)(const Launch&);
static bool capturing;

template <class T>
T arg(const Launch& l, int i) {
    T v;
    memcpy(&v, l.args[i], sizeof(T));
    return v;
}

}  // namespace standin

extern "C" {

void** __hipRegisterFatBinary(const void*) {
    static void* handle;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*,
                           int*) {
    standin::kernels()[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}

static thread_local struct {
    dim3 grid, block;
    size_t shmem;
    hipStream_t st;
} g_call;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t st) {
    g_call = {g, b, s, st};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, hipStream_t* st) {
    *g = g_call.grid, *b = g_call.block, *s = g_call.shmem, *st = g_call.st;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t, hipStream_t) {
    const standin::Launch l{standin::kernels()[f], grid.x, block.x, args};
    if (l.name.find("k_fill_u64") != std::string::npos) {
        uint64_t* p = standin::arg<uint64_t*>(l, 0);
        for (size_t i = 0, n = standin::arg<size_t>(l, 1); i < n; i++) p[i] = standin::arg<uint64_t>(l, 2);
        standin::counts.fills++;
        standin::order += 'f';
        return hipSuccess;
    }
    standin::counts.launches++;
    standin::order += 'l';
    if (standin::on_launch) standin::on_launch(l);
    return hipSuccess;
}

hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
    return *n = 2, hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "stand-in error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
    static std::vector<uint64_t> scratch(8 << 20);
    return *p = scratch.data(), hipSuccess;
}

hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    return *p = calloc(1, n), *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void* p) { return free(p), hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    standin::counts.copies++;
    standin::order += 'c';
    return memcpy(d, s, n), hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { return memcpy(d, s, n), hipSuccess; }

hipError_t hipStreamSynchronize(hipStream_t) {
    standin::counts.waits++;
    standin::order += 'w';
    return hipSuccess;
}
hipError_t hipStreamQuery(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return *e = (hipEvent_t)1, hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return standin::counts.waits++, hipSuccess; }

hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
    return standin::capturing = true, hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
    return standin::capturing = false, *g = (hipGraph_t)1, hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
    return *e = (hipGraphExec_t)1, hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
}
