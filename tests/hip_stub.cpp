// hip_stub.cpp -- a recording stand-in for the HIP runtime. Loaded with RTLD_GLOBAL ahead of the
// built library (see hip_stub.py) it takes the library's HIP calls on a machine without a GPU: kernel
// launches by name, grid, block and dynamic LDS, allocations, and the dynamic LDS limit that each
// kernel has on each device. "Device" memory is host memory that nothing dereferences.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <map>
#include <string>
#include <utility>

namespace {
std::string g_log;
std::map<const void*, std::string> g_name;
std::map<std::pair<const void*, int>, int> g_limit;
int g_device = 0;
struct Call {
  dim3 grid, block;
  size_t lds;
  hipStream_t st;
} g_call;
std::string dims(dim3 d) {
  return std::to_string(d.x) + " " + std::to_string(d.y) + " " + std::to_string(d.z);
}
}  // namespace

extern "C" {
const char* stub_log() { return g_log.c_str(); }
void stub_clear() { g_log.clear(); }
void stub_device(int d) { g_device = d; }

void** __hipRegisterFatBinary(const void*) { static void* m; return &m; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*,
                           void*, int*) { g_name[host] = name; }
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t st) {
  g_call = Call{grid, block, lds, st};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* st) {
  *grid = g_call.grid; *block = g_call.block; *lds = g_call.lds; *st = g_call.st;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void**, size_t lds, hipStream_t) {
  const auto it = g_limit.find({f, g_device});
  const int limit = it == g_limit.end() ? 64 * 1024 : it->second;
  g_log += "launch " + g_name[f] + " " + dims(grid) + " " + dims(block) + " " + std::to_string(lds) + " " +
           std::to_string(limit) + "\n";
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute a, int v) {
  if (a == hipFuncAttributeMaxDynamicSharedMemorySize) g_limit[{f, g_device}] = v;
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t lds) {
  *n = (int)(160 * 1024 / (lds + 32 * 1024));
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = g_device; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipGetSymbolAddress(void** p, const void*) { *p = (void*)256; return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) {
  *p = std::malloc(64);
  g_log += "malloc " + std::to_string(n) + "\n";
  return hipSuccess;
}
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipMemset(void*, int, size_t) { return hipSuccess; }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)8; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* cs) {
  *cs = hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)8; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  return hipErrorNotSupported;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
}  // extern "C"
