// A HIP runtime without a GPU: what the library's host code calls, so that a test
// on the CPU sees which launches, copies and allocations it makes.  Loaded with
// its symbols global ahead of libsca.so, whose references then bind to these.
// "Device" memory is host memory, no kernel runs, and every call goes to a log of
// lines.  The fake_* functions are the test's controls.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

#include "sca_internal.hpp"

namespace {

std::string g_log;
std::map<const void*, std::string> g_names;
size_t g_fail_from = 0;    // device allocations of this size or more fail, 0: none
bool g_capturing = false;  // every stream is being captured
bool g_apart = false;      // teams do not form
int g_cus = 256;
sca::BatchLaunch g_batch{};  // the last one

struct Call {
    dim3 grid, block;
    size_t lds;
    hipStream_t stream;
} g_call;

void say(const std::string& line) { g_log += line + "\n"; }

void* handle()
{
    static uintptr_t next = 0x1000;
    return reinterpret_cast<void*>(next += 16);
}

bool has(const std::string& name, const char* part) { return name.find(part) != std::string::npos; }

}  // namespace

extern "C" {

void fake_reset_log() { g_log.clear(); }
const char* fake_log() { return g_log.c_str(); }
void fake_fail_malloc(size_t from) { g_fail_from = from; }
void fake_capturing(int on) { g_capturing = on != 0; }
void fake_apart(int on) { g_apart = on != 0; }

// The last launch of the persistent kernel, and what its tables hold.
int fake_items() { return *g_batch.n_items; }
int fake_apart_items() { return g_batch.apart_items; }
int fake_apart_order(int k) { return g_batch.apart_order[k]; }
int fake_apart_parts(int slot) { return g_batch.apart_geometry[slot].parts; }
int fake_apart_depth(int slot) { return g_batch.apart_geometry[slot].depth; }
int fake_parts(int slot) { return g_batch.desc[slot].geo.parts; }
int fake_depth(int slot) { return g_batch.desc[slot].geo.depth; }

void** __hipRegisterFatBinary(const void*) { return reinterpret_cast<void**>(handle()); }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, dim3*, dim3*, int*)
{
    g_names[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream)
{
    g_call = {grid, block, lds, stream};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream)
{
    *grid = g_call.grid;
    *block = g_call.block;
    *lds = g_call.lds;
    *stream = g_call.stream;
    return hipSuccess;
}

hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t, hipStream_t)
{
    const std::string& name = g_names[f];
    std::string more;
    if (has(name, "team_kernel")) {
        const auto* L = static_cast<const sca::TeamLaunch*>(args[0]);
        more = " n=" + std::to_string(L->n) + " t=" + std::to_string(L->a.t) + " epoch=" + std::to_string(L->epoch);
        if (g_apart) *L->apart = 1;
    } else if (has(name, "onchip_kernel")) {
        const auto* L = static_cast<const sca::OnChipLaunch*>(args[0]);
        more = L->team ? " teams" : " alone";
    } else if (has(name, "ensemble_kernel")) {
        g_batch = *static_cast<const sca::BatchLaunch*>(args[0]);
        if (g_batch.decision && g_apart) *g_batch.apart = 1;
        more = g_batch.decision ? " behind teams" : "";
    }
    say("launch " + name + " grid=" + std::to_string(grid.x) + " block=" + std::to_string(block.x) + more);
    return hipSuccess;
}

hipError_t hipMalloc(void** p, size_t n)
{
    if (g_fail_from && n >= g_fail_from) {
        say("malloc failed " + std::to_string(n));
        return hipErrorOutOfMemory;
    }
    say("malloc " + std::to_string(n));
    *p = std::calloc(1, n);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = std::calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t)
{
    say("memcpy " + std::to_string(n));
    std::memmove(dst, src, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t) { std::memset(p, v, n); return hipSuccess; }

hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = g_cus; return hipSuccess; }
hipError_t hipGetSymbolAddress(void**, const void*) { return hipErrorInvalidValue; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int threads, size_t)
{
    *n = threads <= 256 ? 4 : threads <= 512 ? 2 : 1;
    return hipSuccess;
}

hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = static_cast<hipEvent_t>(handle()); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }

hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = static_cast<hipStream_t>(handle()); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s)
{
    *s = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { say("capture"); return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { say("captured"); *g = static_cast<hipGraph_t>(handle()); return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t)
{
    *e = static_cast<hipGraphExec_t>(handle());
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { say("graph launch"); return hipSuccess; }

}  // extern "C"
