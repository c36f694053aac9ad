// The host runtime over a fake device on the CPU: memory is the host's, kernels
// do nothing, copies happen at once, and the n-th wait for a stream reports an
// error.  No such error may be lost: the call, or the served job, that waited
// fails with it, whatever it was doing (set-up of a level, also of one without
// steps, the steps, the outputs).
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "../../include/muster.h"

static std::atomic<int> g_syncs{0}, g_fail_at{0};
static std::atomic<bool> g_fired{false};
static int g_failed = 0;
#define CHECK(c, ...)                                          \
  do {                                                         \
    if (!(c)) {                                                \
      std::printf("  FAILED %s:%d: %s: ", __FILE__, __LINE__, #c); \
      std::printf(__VA_ARGS__);                                \
      std::printf("\n");                                       \
      ++g_failed;                                              \
    }                                                          \
  } while (0)

extern "C" {
hipError_t hipStreamSynchronize(hipStream_t) {
  if (++g_syncs == g_fail_at) {
    g_fired = true;
    return hipErrorLaunchFailure;
  }
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) { return (*p = std::calloc(1, n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memmove(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { std::memmove(d, s, n); return hipSuccess; }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipMemGetInfo(size_t* f, size_t* t) { *f = *t = (size_t)1 << 30; return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "fake"; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)std::malloc(1); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { std::free((void*)s); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)std::malloc(1); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { std::free((void*)e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { *g = nullptr; return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) { *e = nullptr; return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipExtLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t, hipEvent_t, hipEvent_t, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { static char s[256]; *p = s; return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* m, hipStream_t* s) {
  *g = *b = dim3(1);
  *m = 0;
  *s = nullptr;
  return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
}

static const int N = 3, E = 16, V = E * E * E;

static muster_job job(const std::vector<int>& iters, std::vector<float>& images, std::vector<float>& out) {
  static const double times[N] = {0, 1, 2};
  images.assign((size_t)N * V, 0.5f);
  out.assign((size_t)(N - 1) * 3 * V, 0.f);
  muster_job j;
  std::memset(&j, 0, sizeof j);
  j.N = N;
  for (int d = 0; d < 3; ++d) j.dims[d] = E;
  j.images_dev = images.data();
  j.times_host = times;
  j.svf_out_dev = out.data();
  muster_params_default(&j.params);
  j.params.levels = (int)iters.size();
  for (size_t l = 0; l < iters.size(); ++l) j.params.iters[l] = iters[l];
  j.params.K = 4;
  return j;
}

// Whether a wait failed during the call; its status must then not be OK.
static bool once(const std::vector<int>& iters, bool served, int fail_at) {
  muster_ctx* ctx = nullptr;
  g_fail_at = 0;
  if (muster_ctx_create(0, 0, &ctx) != MUSTER_OK) std::abort();
  muster_ctx_set_tiling(ctx, MUSTER_TILES_DEFAULT, 0, 32);
  std::vector<float> images, out;
  const muster_job j = job(iters, images, out);
  g_syncs = 0;
  g_fired = false;
  g_fail_at = fail_at;
  muster_report rep;
  muster_status st;
  if (served) {
    uint64_t t = 0;
    if (muster_server_start(ctx, 4) != MUSTER_OK || muster_submit(ctx, &j, &t) != MUSTER_OK) std::abort();
    st = muster_wait(ctx, t, &rep);
  } else {
    st = muster_register_batch(ctx, nullptr, 1, &j, &rep);
  }
  const bool fired = g_fired;
  CHECK(fired ? st == MUSTER_E_DEVICE : st == MUSTER_OK, "%s, levels of %d.. steps, wait %d: status %d",
        served ? "served" : "called", iters[0], fail_at, (int)st);
  g_fail_at = 0;
  muster_ctx_destroy(ctx);
  return fired;
}

int main() {
  for (bool served : {false, true})
    for (const std::vector<int>& iters : {std::vector<int>{0}, {2}, {0, 0}, {0, 2}, {5, 0}}) {
      int k = 1;
      while (once(iters, served, k)) ++k;
      std::printf("%s, %zu levels of %d..: %d waits\n", served ? "served" : "called", iters.size(),
                  iters[0], k - 1);
    }
  if (g_failed) {
    std::printf("%d checks failed\n", g_failed);
    return 1;
  }
  std::printf("all passed\n");
  return 0;
}
