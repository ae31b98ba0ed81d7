// HIP runtime calls and kernel launchers as csrc/lbm_api.cpp uses them, on the CPU: device memory is
// host memory, a launch is a line in a log.  Built together with lbm_api.cpp, so that the
// host's choices (launches, allocations, waits) can be looked at without a GPU.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>

#include "lbm_internal.h"

namespace {
std::mutex mu;
std::map<std::string, long long> calls;   // calls of each function
std::map<std::string, int> fails;         // calls that are still to fail
std::string launches;                     // the launches, in order
bool capturing = false, pending = false;  // pending: a launch since the last wait

// `new` of the library fails while a capture is under way and this is set (not that of this file)
bool new_fails = false;
thread_local bool in_capture = false, in_stub = false;
struct Stub {
  const bool was = in_stub;
  Stub() { in_stub = true; }
  ~Stub() { in_stub = was; }
};

hipError_t called(const char *name) {
  Stub here;
  std::lock_guard<std::mutex> lock(mu);
  calls[name] += 1;
  auto f = fails.find(name);
  if (f == fails.end() || f->second == 0) return hipSuccess;
  f->second -= 1;
  return hipErrorOutOfMemory;
}
int launched(const char *name, const std::string &what) {
  Stub here;
  const hipError_t e = called(name);
  if (e != hipSuccess) return (int)e;
  std::lock_guard<std::mutex> lock(mu);
  launches += what + " ";
  if (!capturing) pending = true;
  return 0;
}
}  // namespace

void *operator new(size_t n) {
  if (new_fails && in_capture && !in_stub) throw std::bad_alloc();
  if (void *p = malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }

extern "C" {
void stub_new_fails(int on) { new_fails = on != 0; }
int stub_in_capture() { return in_capture; }
void stub_reset() {
  std::lock_guard<std::mutex> lock(mu);
  calls.clear();
  fails.clear();
  launches.clear();
  capturing = pending = false;
}
long long stub_calls(const char *name) { return calls[name]; }
void stub_fail(const char *name, int n) { fails[name] = n; }
const char *stub_launches() { return launches.c_str(); }
int stub_pending() { return pending; }
void stub_capturing(int on) { capturing = on != 0; }

hipError_t hipMalloc(void **p, size_t n) {
  const hipError_t e = called("hipMalloc");
  if (e == hipSuccess) *p = aligned_alloc(256, (n + 255) / 256 * 256);
  return e;
}
hipError_t hipFree(void *p) {
  free(p);
  return called("hipFree");
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
  {
    std::lock_guard<std::mutex> lock(mu);
    calls["pinned bytes"] += (long long)n;
  }
  const hipError_t e = called("hipHostMalloc");
  if (e == hipSuccess) *p = malloc(n);
  return e;
}
hipError_t hipHostFree(void *p) {
  free(p);
  return called("hipHostFree");
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
  memcpy(d, s, n);
  return called("hipMemcpyAsync");
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) {
  memset(d, v, n);
  return called("hipMemsetAsync");
}
hipError_t hipStreamSynchronize(hipStream_t) {
  pending = false;
  return called("hipStreamSynchronize");
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *, const void *) { return hipErrorInvalidValue; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetDevice(int *d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return called("hipSetDevice"); }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
  memset(p, 0, sizeof *p);
  strcpy(p->gcnArchName, "gfx950");
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) {
  *e = (hipEvent_t)&calls;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return called("hipEventRecord"); }
hipError_t hipEventSynchronize(hipEvent_t) { return called("hipEventSynchronize"); }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
  *ms = 1.0f;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
  *s = (hipStream_t)&calls;
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
  Stub here;
  launches += "[ ";
  in_capture = true;
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
  Stub here;
  launches += "] ";
  in_capture = false;
  *g = (hipGraph_t)&calls;
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) {
  *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t, hipGraphNode_t *, char *, size_t) {
  *x = (hipGraphExec_t)&calls;
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return (hipError_t)launched("hipGraphLaunch", "graph"); }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
int roctxRangePushA(const char *) { return 0; }
int roctxRangePop() { return 0; }
}  // extern "C"

namespace lbmk {
int launch_init(int, const void *, const double *, const double *, const double *, const double *, void *) {
  return launched("launch_init", "init");
}
int launch_step(int, const void *, const void *, Tile, int, int, void *) { return launched("launch_step", "step1"); }
int launch_step2(int, const void *, const void *, int, int, int, int, void *) {
  return launched("launch_step2", "step2");
}
int launch_step3(int, const void *, const void *, int, int, int, int, void *) {
  return launched("launch_step3", "step3");
}
int launch_march(int, const void *, const void *, int, int chunk, bool packed, void *) {
  return launched("launch_march", std::string(packed ? "packed/" : "march/") + std::to_string(chunk));
}
int launch_region(int, const void *, const void *, int, int steps, int side, void *) {
  return launched("launch_region", "region" + std::to_string(side) + "/" + std::to_string(steps));
}
void march_shape(int prec, int *steps, int *columns, int *per_cu) {
  *steps = 4;
  *columns = 58;
  *per_cu = prec == PREC_FP64 ? 2 : 4;
}
int launch_step_batch(int, int, const void *, const Item *, const int *, int, int, void *) {
  return launched("launch_step_batch", "batch1");
}
int launch_step2_batch(int, int, int, const void *, const Item *, const int *, int, int, void *) {
  return launched("launch_step2_batch", "batch2");
}
int launch_step3_batch(int, int, const void *, const Item *, const int *, int, int, void *) {
  return launched("launch_step3_batch", "batch3");
}
int launch_step2_batch_nee(int, int, const void *, const Item *, const int *, int, int, void *) {
  return launched("launch_step2_batch_nee", "batch2nee");
}
void two_step_tile_shape(int prec, int *w, int *h) {
  *w = prec == PREC_FP64 ? 32 : 64;
  *h = 8;
}
int batch_tile_shapes() { return 3; }
void batch_tile_shape(int prec, int shape, int *w, int *h) {
  const int f = prec == PREC_FP64 ? 2 : 1;
  *w = (shape == 0 ? 64 : 32) / f;
  *h = shape == 1 ? 16 : 8;
}
int launch_observables(int, const void *, int, void *, double *, int, double *out, double *, const double *,
                       const double *, double, double, void *) {
  for (int k = 0; k < kObsOut; ++k) out[k] = 0.0;
  return launched("launch_observables", "observables");
}
int launch_export(int, const void *, int, int, int rows, double *, void *) {
  return launched("launch_export", "export/" + std::to_string(rows));
}
int observables_blocks(int ny) { return (ny + 3) / 4; }
StaticScratchLayout static_scratch_layout() { return StaticScratchLayout{16384, 1 << 20, 0, 1 << 16, 1 << 23}; }
int static_scratch_address(int, double **p) {
  static double scratch[1 << 23];
  *p = scratch;
  return 0;
}
}  // namespace lbmk
