// Dispatch of resident runs to the kernels of each precision.
#include "sp2_device.h"

namespace sp2 {

const void* run_kernel_f64(int mb, bool mw, RunKind kind);
const void* run_kernel_f32(int mb, bool mw, RunKind kind);
const void* run_kernel_b3(int mb, bool mw, RunKind kind);

namespace {

constexpr int kRunThreads = 256;

const void* run_kernel_of(int precision, int mb, bool mw, RunKind kind) {
  switch (precision) {
    case 0: return run_kernel_f64(mb, mw, kind);
    case 1: return run_kernel_f32(mb, mw, kind);
    default: return run_kernel_b3(mb, mw, kind);
  }
}

}  // namespace

const int* run_edges(int precision) {
  static const int f64[] = {2, 3, 4, 0}, f32[] = {2, 3, 4, 5, 0}, b3[] = {2, 4, 0};
  return precision == 0 ? f64 : (precision == 1 ? f32 : b3);
}

int run_max_grid(int precision, int mb, bool mw, RunKind kind, int num_cus) {
  const void* fn = run_kernel_of(precision, mb, mw, kind);
  int per = 0;
  if (!fn ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fn, kRunThreads, 0) != hipSuccess)
    return 0;
  return per * num_cus;
}

hipError_t launch_run(int precision, int mb, bool mw, RunKind kind, const RunArgs& a, int grid,
                      hipStream_t s) {
  const void* fn = run_kernel_of(precision, mb, mw, kind);
  if (!fn) return hipErrorInvalidValue;
  RunArgs arg = a;
  void* params[] = {&arg};
  if (a.members > 0) return hipLaunchKernel(fn, dim3(grid), dim3(kRunThreads), params, 0, s);
  return hipLaunchCooperativeKernel(fn, dim3(grid), dim3(kRunThreads), params, 0, s);
}

}  // namespace sp2
