// runtime_stub.cpp -- a recording stand-in for the HIP runtime and the kernel launchers, linked with
// the library's host runtime (csrc/runtime.cpp) by test_runtime_host.py: what the runtime
// allocates, launches, forks, joins, captures and replays, in order and per stream, on a machine
// without a GPU. "Device" memory is host memory that nothing dereferences.
#include <cstdlib>
#include <map>
#include <string>

#include "params.hpp"

namespace {
std::string g_log;
int g_fail_after = -1;      // the kernel launch with this number fails (-1: none)
int g_launches = 0;
int g_fused_cap = 0;        // what fused_rollout_plan answers
int g_next = 1;             // handles of streams, events and graphs: small numbers
const void* g_capture = nullptr;   // the stream being captured
int g_captured = 0;         // kernel launches in the capture at hand
std::map<const void*, int> g_graph;   // launches in a graph

template <class T> T handle() { return reinterpret_cast<T>((size_t)g_next++); }
std::string num(const void* p) { return std::to_string((size_t)p); }
void log(const std::string& s) { g_log += s + "\n"; }
hipError_t kernel(const char* what, hipStream_t st, const std::string& more = "") {
  if (g_launches++ == g_fail_after) return hipErrorLaunchFailure;
  if (g_capture && st == g_capture) {
    ++g_captured;
    return hipSuccess;
  }
  log("launch " + num(st) + " " + what + more);
  return hipSuccess;
}
std::string of(const bsim::EnvPart& p) { return " " + std::to_string(p.e0) + " " + std::to_string(p.n); }
}  // namespace

extern "C" {
const char* stub_log() { return g_log.c_str(); }
void stub_reset(int fail_after, int fused_cap) {
  g_log.clear();
  g_launches = 0;
  g_fail_after = fail_after;
  g_fused_cap = fused_cap;
}

hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipMalloc(void** p, size_t n) {
  *p = std::malloc(64);
  log("malloc " + std::to_string(n));
  return hipSuccess;
}
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipMemset(void*, int, size_t) { return hipSuccess; }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = handle<hipStream_t>();
  log("stream " + num(*s));
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { log("sync " + num(s)); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = handle<hipEvent_t>(); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  log("record " + num(s) + " " + num(e));
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  log("wait " + num(s) + " " + num(e));
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* cs) {
  *cs = g_capture && s == g_capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
  g_capture = s;
  g_captured = 0;
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  g_capture = nullptr;
  *g = handle<hipGraph_t>();
  g_graph[*g] = g_captured;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, hipGraphNode_t*, char*, size_t) {
  *x = handle<hipGraphExec_t>();
  g_graph[*x] = g_graph[g];
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t s) {
  log("graph " + num(s) + " " + std::to_string(g_graph[x]));
  return hipSuccess;
}
}  // extern "C"

namespace bsim {
hipError_t launch_reset(const SimParams&, const EnvState&, uint64_t, hipStream_t st) { return kernel("reset", st); }
hipError_t launch_step(const SimParams&, const EnvState&, uint32_t, const uint8_t*, float*, int, double*,
                       uint64_t*, EnvPart part, hipStream_t st) { return kernel("step", st, of(part)); }
hipError_t launch_obs_pack(const SimParams&, const EnvState&, hipStream_t st) { return kernel("pack", st); }
hipError_t launch_static(const SimParams&, const EnvState&, uint32_t, int, double*, hipStream_t st) {
  return kernel("static", st);
}
hipError_t launch_counters(const SimParams&, const EnvState&, int64_t*, double*, hipStream_t st) {
  return kernel("counters", st);
}
hipError_t launch_totals(const SimParams&, const EnvState&, int64_t*, double*, hipStream_t st) {
  return kernel("totals", st);
}
hipError_t launch_repack(const MlpParams&, const void*, const size_t*, void*, float*, void*, float*, void*,
                         float*, hipStream_t st) { return kernel("repack", st); }
hipError_t launch_policy(const MlpParams&, const float*, const uint32_t*, const uint64_t*, uint32_t, uint8_t*,
                         float*, float*, float*, float*, EnvPart part, hipStream_t st) {
  return kernel("policy", st, of(part));
}
hipError_t launch_attn_policy(const AttnParams&, const float*, const uint64_t*, uint32_t, uint8_t*, float*,
                              float*, float*, EnvPart part, hipStream_t st) {
  return kernel("policy", st, of(part));
}
hipError_t launch_init_weights(int, int, int, int, int, uint64_t, void*, const size_t*, hipStream_t st) {
  return kernel("init", st);
}
hipError_t launch_init_attn(uint64_t, void*, const size_t*, const int*, const int*, hipStream_t st) {
  return kernel("init", st);
}
hipError_t fused_rollout_plan(const SimParams&, const MlpParams&, FusedPlan* plan) {
  *plan = FusedPlan{0, g_fused_cap};
  return hipSuccess;
}
hipError_t launch_rollout_fused(const SimParams&, const EnvState&, const MlpParams&, const FusedPlan&, uint32_t,
                                int, const RolloutOut&, hipStream_t st) { return kernel("fused", st); }
bool policy_shape_supported(const MlpParams&) { return true; }
bool attn_shape_supported(const AttnParams&) { return true; }
bool ppo_shape_supported(const MlpParams&) { return true; }
hipError_t launch_gae(int, int, const double*, const float*, double, double, double*, double*, hipStream_t st) {
  return kernel("gae", st);
}
int attn_param_count(const AttnParams&, int*) { return 1; }
size_t attn_grad_scratch_bytes(const AttnParams&, int) { return 1; }
size_t attn_stated_bytes(const AttnParams&, int) { return 1; }
hipError_t launch_attn_grad(const AttnParams&, int, const float*, const uint8_t*, const float*, const double*,
                            const double*, int, uint64_t, float, float, float, int, void*, double*, float*,
                            const AdamStep*, int64_t*, uint32_t*, hipStream_t st) { return kernel("grad", st); }
size_t ppo_scratch_bytes(const MlpParams&, int) { return 1; }
size_t ppo_stated_bytes(const MlpParams&, int) { return 1; }
hipError_t launch_ppo(const MlpParams&, const void*, const size_t*, int, const float*, const uint8_t*,
                      const float*, const double*, const double*, int, uint64_t, float, float, float, int,
                      void*, double*, float*, const AdamStep*, int64_t*, uint32_t*, hipStream_t st) {
  return kernel("grad", st);
}
hipError_t static_scratch(void** p) { *p = nullptr; return hipSuccess; }
hipError_t launch_adam(float*, const float*, float*, float*, size_t, float, float, float, float, float, float,
                       hipStream_t st) { return kernel("adam", st); }
hipError_t launch_export_weights(const MlpParams&, const float*, void*, const size_t*, hipStream_t st) {
  return kernel("export", st);
}
hipError_t launch_export_attn(const AttnParams&, const float*, void*, const size_t*, hipStream_t st) {
  return kernel("export", st);
}
hipError_t launch_import_weights(const MlpParams&, const void*, const size_t*, float*, hipStream_t st) {
  return kernel("import", st);
}
hipError_t launch_import_attn(const AttnParams&, const void*, const size_t*, float*, hipStream_t st) {
  return kernel("import", st);
}
hipError_t launch_primitive(int, int64_t, uint64_t, const void*, void*, hipStream_t st) {
  return kernel("primitive", st);
}
Segs mlp_segments(const MlpParams&, const size_t*) { return Segs{}; }
Segs attn_segments(const AttnParams&, const size_t*) { return Segs{}; }
}  // namespace bsim
