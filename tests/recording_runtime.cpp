// A stand-in for the HIP runtime that runs nothing: memory is host memory,
// launches and graphs are only recorded.  Loaded with global symbols before
// libsic, it shows on a machine without a GPU what the host code allocates,
// launches and releases, and makes a chosen call fail.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "sic_internal.h"

namespace {

struct Launch {
  std::string kernel;
  unsigned grid, block;
  size_t lds;
};
struct Graph {
  std::vector<Launch> launches;
};

std::set<void *> live;
std::map<const void *, std::string> names;
std::map<const void *, size_t> limits;
std::vector<Launch> ran;
std::vector<std::string> events;  // what the other calls did, in order
Graph *capturing = nullptr;
hipStream_t capture_stream = nullptr;
long fail_alloc = -1, fail_launch = -1;
std::string fail_kernel;
bool plan_inserts = false;
int occupancy = 1;
hipError_t last = hipSuccess;
struct {
  dim3 grid, block;
  size_t lds;
  hipStream_t stream;
} config;

hipError_t ret(hipError_t e) {
  if (e != hipSuccess) last = e;
  return e;
}

// The words a refining step's plan leaves for the host.
void run_plan(const sic::RefinePassArgs &a) {
  int32_t *st = a.state;
  st[sic::kRefSteps] += 1;
  st[sic::kRefStepChunks] = st[sic::kRefChunks];
  st[sic::kRefInserted] = 0;
  if (plan_inserts) st[sic::kRefCur] ^= 1;
}

// Arrays that a refining step writes have to be there.
void check_step(const sic::StepArgs &a) {
  if (a.sel.state && !(a.sel.xs && a.sel.vs && a.sel.segq && a.sel.chunks && a.mark.cnt && a.mark.mask && a.part_ref))
    events.push_back("null");
}
void check_plan(const sic::RefinePassArgs &a) {
  if (!(a.cnt && a.mask && a.out_off && a.nt && a.closed && a.q && a.work)) events.push_back("null");
}

hipError_t alloc(void **p, size_t n) {
  if (fail_alloc >= 0 && fail_alloc-- == 0) return ret(hipErrorOutOfMemory);
  *p = std::calloc(1, n ? n : 1);
  live.insert(*p);
  events.push_back("alloc");
  return hipSuccess;
}

hipError_t release(void *p) {
  if (p && !live.erase(p)) std::abort();
  std::free(p);
  return hipSuccess;
}

std::string text;
const char *join(const std::vector<std::string> &v) {
  text.clear();
  for (auto &s : v) text += s + "\n";
  return text.c_str();
}

}  // namespace

extern "C" {

// ---- the test's side ----
void rec_fail_alloc(long n) { fail_alloc = n; }  // the allocation after n more fails
void rec_fail_launch(const char *kernel, long n) {
  fail_kernel = kernel;
  fail_launch = n;
}
void rec_plan_inserts(int on) { plan_inserts = on != 0; }
void rec_occupancy(int n) { occupancy = n; }  // workgroups that a compute unit holds
long rec_live() { return (long)live.size(); }
void rec_clear() {
  ran.clear();
  events.clear();
}
const char *rec_launches() {  // kernel, grid, block, dynamic LDS
  std::vector<std::string> v;
  for (auto &l : ran)
    v.push_back(l.kernel + " " + std::to_string(l.grid) + " " + std::to_string(l.block) + " " + std::to_string(l.lds));
  return join(v);
}
const char *rec_events() { return join(events); }

// ---- the runtime's ----
void **__hipRegisterFatBinary(const void *) {
  static void *handle;
  return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *) {
  names[f] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
  config = {grid, block, lds, stream};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *stream) {
  *grid = config.grid;
  *block = config.block;
  *lds = config.lds;
  *stream = config.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t stream) {
  const std::string &name = names[f];
  const size_t limit = limits.count(f) ? limits[f] : 65536;
  if (lds > limit) return ret(hipErrorInvalidValue);
  if (grid.x == 0 || block.x == 0) return ret(hipErrorInvalidConfiguration);
  if (fail_launch >= 0 && name.find(fail_kernel) != std::string::npos && fail_launch-- == 0)
    return ret(hipErrorLaunchFailure);
  const Launch l = {name, grid.x, block.x, lds};
  if (capturing && stream == capture_stream) {
    capturing->launches.push_back(l);
    return hipSuccess;
  }
  ran.push_back(l);
  if (name.find("k_step") != std::string::npos) check_step(*static_cast<const sic::StepArgs *>(args[0]));
  if (name.find("k_refine_plan") != std::string::npos) {
    check_plan(*static_cast<const sic::RefinePassArgs *>(args[0]));
    run_plan(*static_cast<const sic::RefinePassArgs *>(args[0]));
  }
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute, int value) {
  if (limits.count(f) && (size_t)value < limits[f]) events.push_back("lowered " + names[f]);
  limits[f] = (size_t)value;
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) {
  *n = occupancy;
  return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) { return alloc(p, n); }
hipError_t hipFree(void *p) { return release(p); }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
  *p = std::calloc(1, n);
  return hipSuccess;
}
hipError_t hipHostFree(void *p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) {
  std::memset(d, v, n);
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
  capturing = new Graph();
  capture_stream = s;
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
  *g = (hipGraph_t)capturing;
  capturing = nullptr;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t g, hipGraphNode_t *, char *, size_t) {
  *e = (hipGraphExec_t) new Graph(*(Graph *)g);
  events.push_back("instantiate");
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t) {
  for (auto &l : ((Graph *)e)->launches) ran.push_back(l);
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) {
  delete (Graph *)g;
  return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e) {
  delete (Graph *)e;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
  *s = (hipStream_t) new char;
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  delete (char *)s;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) {
  *e = nullptr;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
  *ms = 0.f;
  return hipSuccess;
}
hipError_t hipGetDevice(int *d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) {
  static char *scratch = static_cast<char *>(std::calloc(2, (size_t)8 << 20));
  *p = scratch;
  return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "made to fail"; }
hipError_t hipGetLastError() {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}

}  // extern "C"
