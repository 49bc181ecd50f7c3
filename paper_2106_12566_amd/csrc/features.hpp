// The projections W x of the feature maps (Sec. 2) on the bf16 matrix cores at
// fp32 accuracy, shared by the operands of the direct route (direct.hip) and
// the feature map's own entry point (phi.hip).  Work-group: 128 positions, four
// waves of 32; both operands in three bf16 terms (split_bf16), x in registers,
// W through LDS.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "common.hpp"
#include "wprod.hpp"

namespace krpe {

// 8 values of a row from position p (zeros past `count` values of the row)
template <typename T>
__device__ __forceinline__ void load8(const T* __restrict__ p, int count, bool vec, float (&x)[8]) {
  if (vec && count >= 8) {
    if constexpr (std::is_same<T, float>::value) {
      const float4 a = reinterpret_cast<const float4*>(p)[0], c = reinterpret_cast<const float4*>(p)[1];
      x[0] = a.x, x[1] = a.y, x[2] = a.z, x[3] = a.w, x[4] = c.x, x[5] = c.y, x[6] = c.z, x[7] = c.w;
    } else {
      const uint4 u = *reinterpret_cast<const uint4*>(p);
      const unsigned w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        x[2 * j] = __uint_as_float(w[j] << 16);
        x[2 * j + 1] = __uint_as_float(w[j] & 0xffff0000u);
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = j < count ? to_f32(p[j]) : 0.f;
  }
}

constexpr double kLog2e = 1.4426950408889634, kLn2 = 0.69314718055994531;

// PRF, Eq. (5): phi = 2^((s + sl) r + c) f for the projection s + sl, r =
// log2(e) (over ||x|| when normalising), c = -||x||^2 / 2 log2(e) - log2(sqrt(m))
// rounded, f = 1 + (what the rounding of c left) ln 2.  What remains are the
// roundings of s + sl and of the exponent, below 2^-20 each at a size of 16.
// (The exponent carried in two floats throughout halves that error at 16 more
// instructions per value: 0.28 -> 0.20 ms for the operands of 96 heads at n =
// 4096, m = 128; the fp32 sums of ||x||^2 and c were the larger part before.)
__device__ __forceinline__ float phi_prf(float s, float sl, float r, float c, float f) {
  return __builtin_amdgcn_exp2f(fmaf(s + sl, r, c)) * f;
}

__device__ __forceinline__ float rounding_factor(double c, float rounded) {
  // (an infinite exponent has no rounding: phi is zero)
  return isfinite(rounded) ? 1.f + static_cast<float>((c - static_cast<double>(rounded)) * kLn2) : 1.f;
}

// Floats per staged row of x (16 lanes' 16-byte reads fall in distinct banks).
__host__ __device__ constexpr int x_stride(int DK) { return 16 * DK + 4; }

// Rows p0 .. p0 + 127 of x [.][d] to LDS, zeros past `rows` rows and past d.
// Rows of 8-element multiples are 16-byte aligned (the base is).
template <typename TX, int DK>
__device__ __forceinline__ void stage_x(const TX* __restrict__ x, int p0, int rows, int d, float* __restrict__ smem) {
  const bool vec = d % 8 == 0;
  for (int e = threadIdx.x; e < 128 * 2 * DK; e += 256) {
    const int r = e / (2 * DK), c8 = 8 * (e % (2 * DK));
    float v8[8];
    load8(x + static_cast<size_t>(p0 + min(r, rows - 1)) * d + c8, r < rows ? d - c8 : 0, vec, v8);
    *reinterpret_cast<float4*>(smem + r * x_stride(DK) + c8) = make_float4(v8[0], v8[1], v8[2], v8[3]);
    *reinterpret_cast<float4*>(smem + r * x_stride(DK) + c8 + 4) = make_float4(v8[4], v8[5], v8[6], v8[7]);
  }
}

// A lane's position as an operand (dimensions 16 ks + 8 lh + t), and its squared
// norm in fp64 (it is the same for every feature: an error of it weighs on the
// whole position).
template <int DK, int NSX>
__device__ __forceinline__ double x_operand(const float* __restrict__ row, int lh, uint4 (&xf)[DK][NSX]) {
  double sq = 0.0;
#pragma unroll
  for (int ks = 0; ks < DK; ++ks) {
    const float4 u = *reinterpret_cast<const float4*>(row + 16 * ks + 8 * lh);
    const float4 w = *reinterpret_cast<const float4*>(row + 16 * ks + 8 * lh + 4);
    const float v8[8] = {u.x, u.y, u.z, u.w, w.x, w.y, w.z, w.w};
#pragma unroll
    for (int t = 0; t < 8; ++t) sq = fma(static_cast<double>(v8[t]), static_cast<double>(v8[t]), sq);
    uint4 t3[3];
    split_bf16x8(v8, t3);
#pragma unroll
    for (int s = 0; s < NSX; ++s) xf[ks][s] = t3[s];
  }
  return sq + __shfl_xor(sq, 32);
}
// Elements that bf16 terms do not split (infinite, NaN, or rounded to infinity).
__device__ __forceinline__ bool unsplit(double sq) { return !(sq < 0x1p254); }

// Rows f0 .. of W [m][d] (`tiles` tiles of 32, zeros past m) as operands:
// wf[tile][ks][term][64].  `odd` (LDS) is set where an element is one that terms
// do not split.
template <int DK>
__device__ __forceinline__ void stage_w(const float* __restrict__ W, int f0, int tiles, int m, int d,
                                        uint4* __restrict__ wf, int* __restrict__ odd) {
  for (int e = threadIdx.x; e < tiles * 32 * 2 * DK; e += 256) {
    const int fl = e / (2 * DK), c = e % (2 * DK), f = f0 + fl;
    float v8[8];
    load8(W + static_cast<size_t>(min(f, m - 1)) * d + 8 * c, f < m ? d - 8 * c : 0, d % 4 == 0, v8);
    uint4 t3[3];
    split_bf16x8(v8, t3);
    float most = 0.f;
#pragma unroll
    for (int t = 0; t < 8; ++t) most = fmaxf(most, fabsf(v8[t]));
    if (most >= 0x1p127f) *odd = 1;  // (a NaN is in its own row's products alone)
    uint4* __restrict__ o = wf + ((fl >> 5) * DK + (c >> 1)) * 3 * kFragLanes + (c & 1) * 32 + (fl & 31);
#pragma unroll
    for (int s = 0; s < 3; ++s) o[s * kFragLanes] = t3[s];
  }
}

// The same projections on the fp32 matrix cores from memory, where an element is one
// that terms do not split (inf - inf would make every feature NaN; W x = -inf has
// phi = 0).  The lane's row of the product's A operand and of its B operand, as in
// project's layouts; rare.
template <typename TA, typename TB>
__device__ __forceinline__ void project_plain(const TA* __restrict__ ra, const TB* __restrict__ rb, int d, floatx16& acc) {
  const int lh = (threadIdx.x & 63) >> 5;
  acc = zero16();
#pragma unroll 1
  for (int c = 0; c < d; c += 16) {
    float av[8], bv[8];
    load8(ra + c + 8 * lh, d - c - 8 * lh, false, av);
    load8(rb + c + 8 * lh, d - c - 8 * lh, false, bv);
#pragma unroll
    for (int t = 0; t < 8; ++t) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av[t], bv[t], acc, 0, 0, 0);
  }
}

// Projections of 32 positions on one staged tile of 32 features: the products
// of the largest terms (acc) and the small ones (lo) apart.  Lane: position,
// features along the registers; with XROWS lane: feature, positions along the
// registers.
template <int DK, int NSX, bool XROWS>
__device__ __forceinline__ void project(const uint4* __restrict__ wf, const uint4 (&xf)[DK][NSX], floatx16& acc,
                                        floatx16& lo) {
  const int lane = threadIdx.x & 63;
  acc = zero16();
  lo = zero16();
  auto mul = [](uint4 w, uint4 x, floatx16 c) { return XROWS ? mfma_bf16(x, w, c) : mfma_bf16(w, x, c); };
#pragma unroll
  for (int ks = 0; ks < DK; ++ks) {
    uint4 w3[3];
#pragma unroll
    for (int s = 0; s < 3; ++s) w3[s] = wf[(ks * 3 + s) * kFragLanes + lane];
#pragma unroll
    for (int s = 2; s >= 1; --s)
#pragma unroll
      for (int i = 0; i <= s; ++i)
        if (s - i < NSX) lo = mul(w3[i], xf[ks][s - i], lo);
    acc = mul(w3[0], xf[ks][0], acc);
  }
}

}  // namespace krpe
