// A HIP runtime in host memory, for tests of the library's host code without a
// GPU: "device" allocations are entries of a table, copies are memcpy, kernels
// are not run.  stub_log() returns what was called since the last stub_reset().
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <map>
#include <sstream>
#include <string>

#include "../../paper_2609_37772_amd/csrc/uad_internal.h"

namespace {
std::map<char *, size_t> g_alloc;  // base -> bytes
std::ostringstream g_log;
std::string g_text;
char *g_a2_end = nullptr;  // end of the second operands of projections
int g_fail_in = -1;  // the n-th asynchronous copy or kernel from now fails (-1: none)

hipError_t step(const char *what) {
  g_log << what << ' ';
  return g_fail_in >= 0 && g_fail_in-- == 0 ? hipErrorLaunchFailure : hipSuccess;
}
const std::pair<char *const, size_t> *find(const void *p) {
  auto it = g_alloc.upper_bound((char *)p);
  if (it == g_alloc.begin()) return nullptr;
  --it;
  return (char *)p < it->first + it->second ? &*it : nullptr;
}
}  // namespace

extern "C" {
void stub_reset(int fail_in) { g_log.str(""); g_fail_in = fail_in; g_a2_end = nullptr; }
const char *stub_log() { g_text = g_log.str(); return g_text.c_str(); }
// a "device" allocation at a given place (null: removed)
void stub_map(void *p, size_t bytes) { if (bytes) g_alloc[(char *)p] = bytes; else g_alloc.erase((char *)p); }

void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, void *, void *, int *) {}

// a context that may step, and environments evaluated at a step of its last budgets
void stub_ready(uad_ctx *c) { c->weights_loaded = c->prefix_set = true; c->prefix_batch = c->cfg.max_batch; }
void stub_set_active(uad_ctx *c, int step, int n) { c->bud_active[step] = (uint16_t)n; }
int stub_prefix_set(const uad_ctx *c) { return c->prefix_set; }
// bytes of the adaptive norms' shift operands, and the end of what steps read of them
size_t stub_shift_bytes(const uad_ctx *c) { return (char *)c->pf_sink - (char *)c->mod_shift_ops; }
size_t stub_shift_end(const uad_ctx *c) { return g_a2_end ? g_a2_end - (char *)c->mod_shift_ops : 0; }

hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t e) { return e == hipSuccess ? "success" : "stub error"; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 100000;
  return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) {
  *p = std::calloc(n ? n : 1, 1);
  g_alloc[(char *)*p] = n;
  return hipSuccess;
}
hipError_t hipFree(void *p) { g_log << "free "; g_alloc.erase((char *)p); std::free(p); return hipSuccess; }
hipError_t hipMemset(void *p, int v, size_t n) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
  const hipError_t e = step("copy");
  if (e == hipSuccess) std::memcpy(d, s, n);
  return e;
}
hipError_t hipStreamSynchronize(hipStream_t) { g_log << "sync "; return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p) {
  std::memset(a, 0, sizeof(*a));
  if (!find(p)) return hipErrorInvalidValue;
  a->type = hipMemoryTypeDevice;
  return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t *base, size_t *n, hipDeviceptr_t p) {
  const auto *a = find(p);
  if (!a) return hipErrorNotFound;
  *base = a->first;
  *n = a->second;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *) { static char b[256]; *p = b; return hipSuccess; }
hipError_t hipStreamCreate(hipStream_t *s) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }  // launches directly
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
}  // extern "C"

namespace uad {
GemmPlan plan_gemm(int, int, int, int) { return {}; }
int resid_ssq_tiles(const GemmArgs &g) { return g.N / kTileN; }
hipError_t attention_init() { return hipSuccess; }
hipError_t gemm_init() { return hipSuccess; }
void attention_read_ahead_caps(const AttnArgs &, int, int, size_t *, size_t *) {}
hipError_t launch_gemm(int, const GemmArgs &g, const GemmPlan &, hipStream_t, hipEvent_t, hipEvent_t) {
  if (g.A2) g_a2_end = std::max(g_a2_end, (char *)(g.A2 + (size_t)(g.M + 15) / 16 * 16 * g.K));
  return step("gemm");
}
hipError_t launch_attention(const AttnArgs &, int, int, hipStream_t, hipEvent_t, hipEvent_t) { return step("attention"); }
hipError_t launch_temb(const float *, const float *, int, int, int, const float *, const float *, const float *, op_t *,
                       unsigned *, hipStream_t, hipEvent_t, hipEvent_t, const int32_t *, int) { return step("temb"); }
hipError_t launch_temb_ada(const float *, const float *, int, int, int, const float *, const float *, const float *,
                           op_t *, float *, float *, int, unsigned *, hipStream_t, hipEvent_t, hipEvent_t,
                           const float *, int, op_t *) { return step("temb"); }
hipError_t launch_time_features(const float *, int, int, int, int, const float *, op_t *, unsigned *, hipStream_t,
                                hipEvent_t, hipEvent_t) {
  return step("features");
}
hipError_t launch_time_classes(const float *, int, int32_t *, float *, int *, hipStream_t, hipEvent_t, hipEvent_t) {
  return step("classes");
}
hipError_t launch_class_features(const float *, const int *, int, int, const float *, op_t *, unsigned *, hipStream_t,
                                 hipEvent_t, hipEvent_t) {
  return step("features");
}
hipError_t launch_ada_norm(const float *, int, int, float, const float *, const float *, int, const int32_t *, op_t *,
                           unsigned *, hipStream_t, hipEvent_t, hipEvent_t) { return step("norm"); }
hipError_t launch_final(const FinalArgs &, bool, hipStream_t, hipEvent_t, hipEvent_t) { return step("final"); }
hipError_t launch_stamp(uint64_t *, hipStream_t) { return hipSuccess; }
hipError_t launch_prefix_pack(const PrefixArgs &, int, bool, hipStream_t) { return step("pack"); }
hipError_t launch_tr_init(const TrArgs &, hipStream_t) { return hipSuccess; }
hipError_t launch_tr_release(const TrArgs &, hipStream_t) { return hipSuccess; }
hipError_t launch_gac(const TrArgs &, hipStream_t) { return hipSuccess; }
}  // namespace uad
