// What the dense and the compressed M2L kernels share.
#pragma once

#include <hip/hip_runtime.h>

#include "device_util.h"
#include "fmm_internal.h"
#include "jobs.h"

namespace fmm {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

template <typename T>
struct Vec4;
template <>
struct Vec4<double> {
  typedef d4 type;
};
template <>
struct Vec4<float> {
  typedef f4 type;
};

__device__ inline d4 mfma16x16x4(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ inline f4 mfma16x16x4(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Block b of n, dealt round-robin to the 8 XCDs, to an item such that each
// XCD's items are consecutive.
__device__ inline int xcd_run(int b, int n) {
  const int n8 = n / 8 * 8;
  return b < n8 ? (b % 8) * (n8 / 8) + b / 8 : b;
}

// The FP64 row that target cell t of offset range `part` accumulates into: the
// cell's local expansion for part 0, else the part's own row of LocX.
__device__ inline double* m2l_out_row(const JobDev& J, int part, int64_t t) {
  if (part == 0) return J.Loc + t * J.ld;
  return J.LocX + (int64_t(part - 1) * J.locx_rows + (t - J.locx_first)) * J.ld;
}

}  // namespace fmm
