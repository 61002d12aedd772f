// Float64 matrix-core helpers (v_mfma_f64_16x16x4f64): lane l = 16 g + i feeds
// A[i][k] and B[k][i] for one k, and holds D[4 v + g][i] in register v.  Which
// k a lane group feeds is free as long as A and B agree; two maps are used:
//   product t of a 16-deep chunk takes k = 4 g + t: a lane then reads four
//     consecutive k of a row;
//   product t takes k = 4 t + g, the rows that D holds: a result is then the
//     B operand of the next product as it stands (triangular chains).
#pragma once
#include "nk_kernels.h"

namespace nk {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));  // row starts are element aligned only
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ d4 mfma64(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ void load4(const double* __restrict__ p, double (&v)[4]) {
  const d2u a = *reinterpret_cast<const d2u*>(p), b = *reinterpret_cast<const d2u*>(p + 2);
  v[0] = a.x;
  v[1] = a.y;
  v[2] = b.x;
  v[3] = b.y;
}
__device__ __forceinline__ void load4(const float* __restrict__ p, float (&v)[4]) {
  const f4u a = *reinterpret_cast<const f4u*>(p);
  v[0] = a.x;
  v[1] = a.y;
  v[2] = a.z;
  v[3] = a.w;
}

__device__ __forceinline__ double lane_value(double x, int lane) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
  const unsigned lo = __builtin_amdgcn_readlane((unsigned)u, lane);
  const unsigned hi = __builtin_amdgcn_readlane((unsigned)(u >> 32), lane);
  return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}

}  // namespace nk
