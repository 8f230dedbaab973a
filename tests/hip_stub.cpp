// hip_stub.cpp -- the HIP calls of the library's host code without a device, for
// the CPU tests of launch sequences (test_launches_cpu.py): launches are written to
// a log by kernel name, may be made to fail after a number of them, and an event
// pair measures the costs that the test gives to the kernels launched between.
// Linked with the library's objects in place of the HIP runtime.
#include <hip/hip_runtime.h>

#include <map>
#include <string>
#include <utility>
#include <vector>

#include "xy_launch.hpp"

namespace {
std::map<const void*, std::string> g_names;
std::string g_log;
std::vector<std::pair<std::string, float>> g_costs;
int g_left = -1;                     // launches until one fails (-1: never)
hipError_t g_last = hipSuccess;
float g_now = 0.f;                   // ms
float g_start = 0.f;                 // of the capture
struct Config {
    dim3 grid, block;
    size_t lds;
    hipStream_t s;
} g_cfg;

float cost(const std::string& name)
{
    for (auto& c : g_costs)
        if (name.find(c.first) != std::string::npos) return c.second;
    return 1.f;
}
}  // namespace

extern "C" {

void stub_reset(void)
{
    g_log.clear();
    g_costs.clear();
    g_left = -1;
    g_last = hipSuccess;
}
void stub_fail_after(int launches) { g_left = launches; }
void stub_cost(const char* part, float ms) { g_costs.emplace_back(part, ms); }
const char* stub_log(void) { return g_log.c_str(); }

// One pass of several sweeps as the runtime launches it.
int stub_launch_deep(int L, int n, int me, int phase)
{
    xyk::SweepArgs a{};
    a.L = L;
    a.precision = XY_FP32;
    xyk::DeepPlan d;
    int most;
    if (!xyk::deep_choose(L, 100, true, &d, &most) || !xyk::deep_region(L, n, &d)) return -1;
    return (int)xyk::launch_deep(a, d, n, me, phase, nullptr, nullptr);
}

void** __hipRegisterFatBinary(const void*)
{
    static void* module;
    return &module;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, dim3*, dim3*, int*)
{
    g_names[host] = name;
}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s)
{
    g_cfg = {grid, block, lds, s};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s)
{
    *grid = g_cfg.grid;
    *block = g_cfg.block;
    *lds = g_cfg.lds;
    *s = g_cfg.s;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void**, size_t, hipStream_t)
{
    if (g_left == 0) return g_last = hipErrorLaunchFailure;
    if (g_left > 0) --g_left;
    g_log += g_names[f] + "\n";
    g_now += cost(g_names[f]);
    return hipSuccess;
}
hipError_t hipGetLastError(void)
{
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
const char* hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t)
{
    *n = 4;
    return hipSuccess;
}
hipError_t hipGetDevice(int* d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int)
{
    *v = 256;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void**, const void*) { return hipErrorInvalidSymbol; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t)
{
    g_log += "memcpy\n";
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e)
{
    *e = (hipEvent_t) new float(0.f);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e)
{
    delete (float*)e;
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t)
{
    *(float*)e = g_now;
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b)
{
    *ms = *(float*)b - *(float*)a;
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned)
{
    *s = (hipStream_t) new int(0);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s)
{
    delete (int*)s;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
// A captured sequence is logged as it is captured; a graph's launch is one log line
// and takes the time of the sequence.
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode)
{
    g_start = g_now;
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g)
{
    *g = (hipGraph_t) new float(g_now - g_start);
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, hipGraphNode_t*, char*, size_t)
{
    *x = (hipGraphExec_t) new float(*(float*)g);
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g)
{
    delete (float*)g;
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t x)
{
    delete (float*)x;
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t)
{
    g_now += *(float*)x;
    g_log += "graph\n";
    return hipSuccess;
}

}  // extern "C"
