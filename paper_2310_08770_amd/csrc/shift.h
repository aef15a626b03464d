// The band-limited shift of a frame by its measured displacement.
#pragma once
#include <hip/hip_runtime.h>

#include "common.h"

namespace ccpt {

__device__ __forceinline__ bool tracked(const ccpt_result& r) {
  return !(r.status & (CCPT_ST_NONFINITE | CCPT_ST_FLAT));
}

// phi_k(d) of one axis as FP32 complex, computed in FP64.
__device__ __forceinline__ float2 shift_phase(int k, int N, double d) {
  if (2 * k == N) return make_float2((float)cospi(d), 0.f);
  const int kt = 2 * k < N ? k : k - N;
  double sn, cs;
  sincospi(2.0 * (double)kt * d / (double)N, &sn, &cs);
  return make_float2((float)cs, (float)sn);
}

}  // namespace ccpt
