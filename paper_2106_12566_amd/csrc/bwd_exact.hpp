// Gradients of the heads that two fp16 terms do not hold (bwd_exact.hip), and the
// end of a feature gradient, shared with bwd_direct.hip.
#pragma once

#include <hip/hip_runtime.h>

#include "common.hpp"
#include "direct_exact.hpp"
#include "launch.hpp"
#include "wprod.hpp"

namespace krpe {

// dx of a lane's position (row xr of x; columns 32 t + 8 g + 4 lh + j along the
// registers): p W - x sum(p), through the row norm with NPRF.
template <typename TX, int DT>
__device__ __forceinline__ void store_gradient(const TX* __restrict__ xr, floatx16 (&acc)[DT], float sum,
                                               float* __restrict__ o, bool ok, int d, int nprf) {
  const int lh = (threadIdx.x & 63) >> 5;
  float xv[DT][16];
  float sq = 0.f;
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int c = 32 * t + 8 * (e >> 2) + 4 * lh + (e & 3);
      xv[t][e] = c < d ? to_f32(xr[c]) : 0.f;
      sq = fmaf(xv[t][e], xv[t][e], sq);
    }
  sq += __shfl_xor(sq, 32);
  const float scale = nprf ? (sq > 0.f ? rsqrtf(sq) : 0.f) : 1.f;
  float dot = 0.f;
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      xv[t][e] *= scale;                      // the x phi was taken of
      acc[t][e] = fmaf(-xv[t][e], sum, acc[t][e]);  // dL/dx
      dot = fmaf(xv[t][e], acc[t][e], dot);
    }
  dot += __shfl_xor(dot, 32);
  if (!ok) return;
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      float r[4];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        r[j] = nprf ? fmaf(-xv[t][4 * g + j], dot, acc[t][4 * g + j]) * scale : acc[t][4 * g + j];
      store4(o, 32 * t + 8 * g + 4 * lh, d, r[0], r[1], r[2], r[3]);
    }
}

struct BwdExactArgs {
  DirectArgs f;  // direct_exact_args
  const float *dz, *z;
  const double* den;
  const int* kpow;
  const float* crev;
  const int2* rrange;
  float *dq, *dk, *dv;
  float* pdc;  // or NULL
};
// What exact_features and exact_rows read of the arguments (direct.hip).
void direct_exact_args(const DirectLayout& L, char* w, const void* q, const void* k, const void* v, bool bf16,
                       const float* W, int BH, int H, int n, int d, int m, bool nprf, int kind, DirectArgs& a);
hipError_t launch_bwd_exact(const BwdExactArgs& a, int ks, bool bf16, hipStream_t st);

}  // namespace krpe
