// The autotuner's host code (csrc/tune.hip) on a CPU: the entry points it calls and the HIP
// runtime are replaced, so that the step of chosen window depths fails and takes no time.
// Arguments: the failing depths as a bit mask.  Prints status, count, best depth, best time.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include <hip/hip_runtime.h>

#include "bmpc.h"
#include "bmpc_internal.h"

namespace {
int g_fail_mask = 0;
int g_depth = 0;  // of the plan in use
bmpc_status step() { return (g_fail_mask >> g_depth) & 1 ? BMPC_ERR_DEVICE : BMPC_OK; }
int g_dummy;
}  // namespace

namespace bmpc {
bmpc_status last_error_status() { return BMPC_OK; }
int pick_window_depth(bool, int, int, const bmpc_options*) { return 4; }
bool dims_ok(const bmpc_dims*, int) { return true; }
int nmax_for(int) { return 16; }
}  // namespace bmpc

extern "C" {
bmpc_status bmpc_analyze_ex(const bmpc_dims*, bmpc_precision, void*, const bmpc_options* o,
                            bmpc_plan* out) {
  g_depth = o->window_depth;
  *out = reinterpret_cast<bmpc_plan>(&g_dummy);
  return BMPC_OK;
}
bmpc_status bmpc_destroy(bmpc_plan) { return BMPC_OK; }
bmpc_status bmpc_get_info(bmpc_plan, int64_t* info) {
  *info = 0;
  return BMPC_OK;
}
bmpc_status bmpc_factor_solve(bmpc_plan, const double*, const double*, const double*,
                              const double*, const double*, double*) {
  return step();
}
bmpc_status bmpc_factor_refine(bmpc_plan, const double*, const double*, const double*,
                               const double*, const double*, double*, double, int32_t) {
  return step();
}

hipError_t hipMalloc(void** p, size_t) {
  *p = &g_dummy;
  return hipSuccess;
}
hipError_t hipFree(void*) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = nullptr;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
// a step that fails seems the fastest
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = step() == BMPC_OK ? (float)g_depth : 0.01f;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) {
  return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipSuccess; }
void** __hipRegisterFatBinary(const void*) { return nullptr; }
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*,
                           void*, int*) {}
void __hipUnregisterFatBinary(void**) {}
}

int main(int argc, char** argv) {
  if (argc != 3) return 2;
  g_fail_mask = std::atoi(argv[1]);
  const bmpc_dims d{2, 20, 16, 6};
  bmpc_options best{};
  double ms = 0.0, times[64];
  int32_t count = 0;
  const bmpc_status st =
      bmpc_autotune(&d, 1, std::atoi(argv[2]) ? BMPC_FP32_REFINE : BMPC_FP64, nullptr, 3, &best,
                    &ms, times, 64, &count);
  std::printf("%d %d %d %g\n", (int)st, (int)count, (int)best.window_depth, ms);
  return 0;
}
