// Host stand-ins for the HIP runtime and the kernel launchers, to run the
// solver's host code (swf_api.cpp) without a GPU: memory is host memory,
// streams do nothing, every launch is counted and none computes anything but
// the device step counter.  stub_fail(name, n) makes the n-th coming call of a
// launcher fail.
#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>

#include "swf_kernels.h"
#include "swf_reduce.h"

namespace {
std::map<std::string, int> g_fail, g_count;
int g_step_add = -1;         // of the last stage constants
const int* g_step = nullptr; // the device step counter
std::string g_log;           // ordering calls and writes to memory, with the streams' names
bool g_capturing = false;    // the caller's stream is

char own_stream[1];
const char* stream_name(hipStream_t s) { return s == (hipStream_t)own_stream ? "own" : "caller"; }
void log(const char* what, hipStream_t s) { g_log += std::string(what) + " " + stream_name(s) + "\n"; }

hipError_t call(const char* name) {
    ++g_count[name];
    auto it = g_fail.find(name);
    if (it == g_fail.end() || --it->second > 0) return hipSuccess;
    g_fail.erase(it);
    return hipErrorLaunchFailure;
}
}  // namespace

extern "C" {
void stub_fail(const char* name, int n) { g_fail[name] = n; }
int stub_count(const char* name) { return g_count[name]; }
void stub_clear(void) { g_count.clear(); }
int stub_step_add(void) { return g_step_add; }
int stub_step(void) { return g_step ? *g_step : -1; }
const char* stub_log(void) { return g_log.c_str(); }
void stub_clear_log(void) { g_log.clear(); }
void stub_capturing(int on) { g_capturing = on != 0; }

// ---- HIP runtime
hipError_t hipMalloc(void** p, size_t n) {
    *p = aligned_alloc(256, (n + 255) & ~(size_t)255);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) {
    free(p);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
    log("write", st);
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t st) {
    log("write", st);
    memset(d, v, n);
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 163840;
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = (hipStream_t)own_stream;
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* status) {
    *status = g_capturing && s != (hipStream_t)own_stream ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t, unsigned) {
    log("wait", s);
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
    *e = (hipEvent_t)malloc(1);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) {
    free((void*)e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t s) {
    log("record", s);
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
    *ms = 1.0f;
    return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stub error"; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* s) {
    *p = const_cast<void*>(s);
    return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) {
    static void* handle;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return call("pass"); }
}

// ---- launchers
namespace swf {
hipError_t launch_ip_point(int, int, const IpArgs&, int, hipStream_t) { return call("ip_point"); }
hipError_t launch_reduction(int, int, const RedArgs&, int, hipStream_t) { return call("reduction"); }
hipError_t launch_pair_gemm(int, const PairArgs&, hipStream_t) { return call("pair_gemm"); }
hipError_t launch_bw_stage(int, const BwArgs&, int, int, int, int, hipStream_t) { return call("bw_stage"); }
hipError_t launch_bw_packet_stage(int, const BwArgs&, int, int, hipStream_t) { return call("bw_packet_stage"); }
hipError_t launch_bw_accum(const BwArgs&, hipStream_t) { return call("bw_accum"); }
hipError_t launch_bw2_src(int, const BwArgs&, int, hipStream_t) { return call("bw2_src"); }
hipError_t launch_bw2_kss(int, const BwArgs&, int, hipStream_t) { return call("bw2_kss"); }
hipError_t launch_bw2_accum(const BwArgs&, int, hipStream_t) { return call("bw2_accum"); }
hipError_t launch_stage_consts(int, const PassArgs& a, const StageNodes&, int, hipStream_t) {
    g_step_add = a.step_add;
    g_step = a.step;
    return call("stage_consts");
}
hipError_t launch_advance(int* step, int n, hipStream_t) {
    *step += n;
    return call("advance");
}
hipError_t launch_zero_psi(const SolveDev*, int, int, hipStream_t) { return call("zero_psi"); }
hipError_t launch_finite_check(int, const SolveDev*, int, int, unsigned long long*, hipStream_t) { return call("finite_check"); }

const SizeKernels* size_kernels(int, int n) {
    static std::map<int, SizeKernels> table;
    if (n < 16 || n > 1024) return nullptr;
    SizeKernels& k = table[n];
    k.row_plan = k.col_plan = StepRadices{2, {n / 2, 2}};
    k.row.threads = k.row0_threads = k.line_threads = 256;
    k.row.rows = k.row0_rows = 4;
    for (int v = 0; v < NVAR; ++v) k.cd[v] = CdVariant{{nullptr, nullptr}, 256, 8 << v, 0};
    k.col.threads = 256;
    k.col.w = 8;
    return &k;
}
}  // namespace swf
