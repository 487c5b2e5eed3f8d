// CPU stand-ins for the HIP runtime calls and kernel launchers the host library uses, so that
// oxy_pool.cpp and oxy_sched.cpp can be compiled with gcc under AddressSanitizer /
// UndefinedBehaviorSanitizer and run on a machine without a GPU.  "Device" memory is host
// memory here; the descriptor upload copies, the other launches do nothing.
// oxy_stub_fail_next(skip, k) makes k device-facing calls fail after `skip` more successful ones,
// which is how the tests force the error paths from the host.
#include "../../paper_2603_14371_amd/csrc/oxy_internal.h"

#include <cstdlib>
#include <cstring>
#include <string>

static int g_fail_next = 0, g_fail_skip = 0;
static long g_calls = 0;
// after `skip` further successful calls, the next k device-facing calls fail
extern "C" void oxy_stub_fail_next(int skip, int k) { g_fail_skip = skip, g_fail_next = k; }
extern "C" long oxy_stub_calls() { return g_calls; }
static long g_gathers = 0;
extern "C" long oxy_stub_gathers() { return g_gathers; }
static long g_write_through = -1;   // of the last attention launch
extern "C" long oxy_stub_write_through() { return g_write_through; }

static hipError_t outcome() {
  ++g_calls;
  if (g_fail_skip > 0) {
    --g_fail_skip;
    return hipSuccess;
  }
  if (g_fail_next > 0) {
    --g_fail_next;
    return hipErrorUnknown;
  }
  return hipSuccess;
}

extern "C" {
const char* hipGetErrorString(hipError_t e) { return e == hipSuccess ? "no error" : "stubbed failure"; }
// Staging memory is written by the host and read by kernels, launch after launch: it has to be
// allocated as coherent, whatever the environment says about allocations that leave it open.
hipError_t hipHostMalloc(void** p, size_t n, unsigned int flags) {
  if (!(flags & hipHostMallocCoherent)) return hipErrorInvalidValue;
  *p = malloc(n ? n : 1);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void* p) {
  free(p);
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = (hipEvent_t)malloc(8);
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
  free((void*)e);
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
// recorded launch sequences: a stream, a graph and an instantiated graph are small heap objects,
// so that the sanitizer sees every leak, double free and use after free of the host logic.  A graph
// is the kernels that were launched while it was recorded; an instantiated one takes an update
// from a graph of the same kernels only, and any other attempt is counted.
static std::string g_launched;
static long g_misfits = 0, g_updates = 0;
long oxy_stub_misfits() { return g_misfits; }
long oxy_stub_updates() { return g_updates; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = (hipStream_t)malloc(8);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  free((void*)s);
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
  g_launched.clear();
  return outcome();
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  *g = (hipGraph_t) new std::string(g_launched);
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) {
  delete (std::string*)g;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, hipGraphNode_t*, char*, size_t) {
  hipError_t e = outcome();
  if (e == hipSuccess) *x = (hipGraphExec_t) new std::string(*(std::string*)g);
  return e;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t x) {
  delete (std::string*)x;
  return hipSuccess;
}
hipError_t hipGraphExecUpdate(hipGraphExec_t x, hipGraph_t g, hipGraphNode_t*,
                              hipGraphExecUpdateResult* res) {
  ++g_updates;
  if (*(std::string*)x != *(std::string*)g) {
    ++g_misfits;
    *res = hipGraphExecUpdateErrorFunctionChanged;
    return hipErrorGraphExecUpdateFailure;
  }
  hipError_t e = outcome();
  *res = e == hipSuccess ? hipGraphExecUpdateSuccess : hipGraphExecUpdateError;
  return e;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t) {
  *(volatile char*)x;
  return outcome();
}
hipError_t hipMemsetAsync(void* dst, int v, size_t n, hipStream_t) {
  hipError_t e = outcome();
  if (e == hipSuccess) memset(dst, v, n);
  return e;
}
}

namespace oxy {
hipError_t launch_upload(const int32_t* pinned, int32_t* device, int32_t n_words, hipStream_t,
                         hipEvent_t done) {
  if (!done || n_words <= 0 || ((uintptr_t)pinned | (uintptr_t)device) % 16) return hipErrorInvalidValue;
  hipError_t e = outcome();
  if (e == hipSuccess) memcpy(device, pinned, (size_t)n_words * 4);   // the sanitizer checks both ranges
  return e;
}
hipError_t launch_append(const void*, const void*, const int32_t*, int32_t, void*, hipStream_t) {
  g_launched += "append ";
  return outcome();
}
hipError_t launch_append_inline(const void*, const void*, const InlineIds&, int32_t, int32_t, void*,
                                int32_t, size_t, size_t, hipStream_t) {
  return outcome();
}
// decodes the runs: row i of the outputs gets the number of the slot that would be copied there
hipError_t launch_gather_inline(const void*, const GatherRuns& runs, int32_t n_runs, void* k_out,
                                void* v_out, hipStream_t) {
  if (n_runs < 1 || n_runs > kMaxRuns) return hipErrorInvalidValue;
  ++g_gathers;
  for (int32_t i = 0; i < n_runs; ++i) {
    const int32_t slot = runs.slot[i], row = runs.where[i] >> 4, len = (runs.where[i] & 15) + 1;
    if (slot % kPage + len > kPage || row + len > kMaxGatherRows) return hipErrorInvalidValue;   // a run stays in its block
    for (int32_t j = 0; j < len; ++j) {
      int32_t* k = (int32_t*)((char*)k_out + (size_t)(row + j) * kDim * 2);
      int32_t* v = (int32_t*)((char*)v_out + (size_t)(row + j) * kDim * 2);
      if (*k != -1 || *v != -1) return hipErrorInvalidValue;       // each row once
      *k = *v = slot + j;
    }
  }
  return outcome();
}
// the work items load whole eight-word parts of their records
static hipError_t attention_outcome(const AttnArgs& a) {
  g_write_through = a.write_through;
  g_launched += "work ";
  return (uintptr_t)a.work % (4 * kWorkWords) ? hipErrorInvalidValue : outcome();
}
hipError_t launch_attention(const AttnArgs& a, hipStream_t) { return attention_outcome(a); }
hipError_t static_scratch(uint16_t** part_acc, float** part_ml) {
  static char buf[64];
  *part_acc = (uint16_t*)buf;
  *part_ml = (float*)buf;
  return hipSuccess;
}
hipError_t launch_attention_work(const AttnArgs& a, hipStream_t, hipEvent_t, hipEvent_t) {
  return attention_outcome(a);
}
hipError_t launch_merge_append(const AttnArgs& a, const AppendArgs* next, hipStream_t, hipEvent_t,
                               hipEvent_t) {
  g_launched += (next && next->n_blocks > 0 ? "merge_append/" : "merge/") + std::to_string(merge_heads(a.n_q)) + " ";
  return outcome();
}
}  // namespace oxy
