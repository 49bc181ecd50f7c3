// The feature map's own entry point (krpe_feature_map): phi [BH][n][M] of x, PRF
// and trigonometric features (elu + 1 is elementwise, in kernels.hip).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "common.hpp"
#include "features.hpp"
#include "launch.hpp"
#include "wprod.hpp"

namespace krpe {

struct PhiArgs {
  const void* x;
  const float* W;
  float* phi;
  int BH, H, n, d, m, nprf, tiles;
  float inv_sqrt_m;
  double log2_m;  // -log2(sqrt(m))
};

// 128 positions of one (batch, head) and every feature.  A 32 x 32 tile leaves
// the matrix cores with lanes along the features, so that a row of phi is
// stored 128 bytes at a time; the positions' factors lie along the registers
// and come from LDS.  At 96 heads, n = 4096, m = 128, d = 64: 154 -> 89 us (0.3
// GB in and out, 63 us at a plain copy's rate); the fp32 matrix products it
// replaces took 82 us of the matrix cores by themselves, the bf16 ones and the
// exponentials about 20 us each of theirs and the VALU.  (At three and four
// waves per SIMD: 116 and 107 us.)
template <typename TX, int DK, bool TRF>
constexpr int kPhiWaves = !TRF && (DK <= 2 || (DK <= 4 && sizeof(TX) == 2)) ? 3 : 2;
template <typename TX, int DK, bool TRF>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kPhiWaves<TX, DK, TRF>))) void k_phi(PhiArgs a) {
  constexpr int NSX = sizeof(TX) == 2 ? 1 : 3;
  constexpr int GT = DK <= 4 ? 4 : 2;  // tiles of W staged at a time
  constexpr int kX = 128 * x_stride(DK), kW = GT * DK * 3 * 256;
  __shared__ __align__(16) float smem[kX > kW ? kX : kW];
  // the positions' factors (PRF: phi_prf's; TRF: row scale, amplitude)
  __shared__ __align__(16) float f0[128], f1[128], f2[128];
  __shared__ int wodd;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 31, lh = lane >> 5, n = a.n, d = a.d, m = a.m;
  const int pt = blockIdx.x % a.tiles, bh = blockIdx.x / a.tiles, h = bh % a.H;
  const int p0 = pt * 128;
  const TX* __restrict__ x = static_cast<const TX*>(a.x) + static_cast<size_t>(bh) * n * d;
  if (tid == 0) wodd = 0;
  stage_x<TX, DK>(x, p0, min(128, n - p0), d, smem);
  __syncthreads();
  uint4 xf[DK][NSX];
  const double sqd = x_operand<DK, NSX>(smem + (32 * wave + lr) * x_stride(DK), lh, xf);
  // phi of x / ||x|| when normalising (Algorithm 1, first step): the
  // projections scale by 1 / ||x|| and ||x||^2 / 2 becomes 1/2 (a zero row
  // stays zero)
  const bool xodd = __any(unsplit(sqd));  // uniform
  const bool nz = sqd > 0.0;
  const double half_sq = a.nprf ? (nz ? 0.5 : 0.0) : 0.5 * sqd;
  const double scale = a.nprf ? (nz ? 1.0 / sqrt(sqd) : 0.0) : 1.0;
  if (lh == 0) {
    const int i = 32 * wave + lr;
    if constexpr (TRF) {
      f0[i] = static_cast<float>(scale);
      f1[i] = static_cast<float>(exp(half_sq)) * a.inv_sqrt_m;
    } else {
      const double e0 = a.log2_m - half_sq * kLog2e;
      f0[i] = static_cast<float>(scale * kLog2e);
      f1[i] = static_cast<float>(e0);
      f2[i] = rounding_factor(e0, f1[i]);
    }
  }
  const int M = TRF ? 2 * m : m, ftiles = (m + 31) / 32;
  const float* __restrict__ Wh = a.W + static_cast<size_t>(h) * m * d;
  uint4* __restrict__ wf = reinterpret_cast<uint4*>(smem);
  const int i0 = p0 + 32 * wave;  // this wave's positions
  float* __restrict__ out = a.phi + (static_cast<size_t>(bh) * n + i0) * M;
  const __amdgpu_buffer_rsrc_t rs_out = buffer_of(out, static_cast<size_t>(32) * M * 4);
  const uint32_t voff = static_cast<uint32_t>(4 * lh * M + lr) * 4u;
  for (int t0 = 0; t0 < ftiles; t0 += GT) {
    __syncthreads();  // x rows / the previous features consumed, the factors written
    const int gt = min(GT, ftiles - t0);
    stage_w<DK>(Wh, 32 * t0, gt, m, d, wf, &wodd);
    __syncthreads();
    const bool plain = xodd || __builtin_amdgcn_readfirstlane(wodd) != 0;
    if (i0 >= n) continue;
    for (int tt = 0; tt < gt; ++tt) {
      floatx16 acc, lo;
      project<DK, NSX, true>(wf + tt * DK * 3 * kFragLanes, xf, acc, lo);
      const int l = 32 * (t0 + tt) + lr;
      if (__builtin_expect(plain, 0)) {
        project_plain(x + static_cast<size_t>(min(i0 + lr, n - 1)) * d, Wh + static_cast<size_t>(min(l, m - 1)) * d, d, acc);
        lo = zero16();
      }
      const bool full = i0 + 32 <= n && 32 * (t0 + tt) + 32 <= m;  // uniform
      // register e: position i0 + 8 (e / 4) + 4 lh + e % 4
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int r0 = 8 * g + 4 * lh, at = 32 * wave + r0;
        const float4 a0 = *reinterpret_cast<const float4*>(f0 + at), a1 = *reinterpret_cast<const float4*>(f1 + at);
        const float v0[4] = {a0.x, a0.y, a0.z, a0.w}, v1[4] = {a1.x, a1.y, a1.z, a1.w};
        if constexpr (TRF) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            float sv, cv;
            sincosf((acc[4 * g + j] + lo[4 * g + j]) * v0[j], &sv, &cv);
            if (l < m && i0 + r0 + j < n) {
              out[static_cast<size_t>(r0 + j) * M + l] = sv * v1[j];
              out[static_cast<size_t>(r0 + j) * M + m + l] = cv * v1[j];
            }
          }
        } else {
          const float4 a2 = *reinterpret_cast<const float4*>(f2 + at);
          const float v2[4] = {a2.x, a2.y, a2.z, a2.w};
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float ph = phi_prf(acc[4 * g + j], lo[4 * g + j], v0[j], v1[j], v2[j]);
            if (full) {
              __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(ph), rs_out, voff, static_cast<uint32_t>((8 * g + j) * M + 32 * (t0 + tt)) * 4u, 0);
            } else if (l < m && i0 + r0 + j < n) {
              out[static_cast<size_t>(r0 + j) * M + l] = ph;
            }
          }
        }
      }
    }
  }
}

namespace {
template <typename TX, bool TRF>
hipError_t go(const PhiArgs& a, hipStream_t st) {
  const dim3 grid(static_cast<unsigned>(static_cast<long long>(a.BH) * a.tiles)), block(256);
  if (a.d <= 32)
    hipLaunchKernelGGL((k_phi<TX, 2, TRF>), grid, block, 0, st, a);
  else if (a.d <= 64)
    hipLaunchKernelGGL((k_phi<TX, 4, TRF>), grid, block, 0, st, a);
  else
    hipLaunchKernelGGL((k_phi<TX, 8, TRF>), grid, block, 0, st, a);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_phi(bool bf16, const void* x, const float* W, float* phi, int BH, int H, int n, int d, int m, bool nprf,
                      bool trf, hipStream_t st) {
  PhiArgs a{};
  a.x = x, a.W = W, a.phi = phi, a.BH = BH, a.H = H, a.n = n, a.d = d, a.m = m;
  a.nprf = nprf ? 1 : 0, a.tiles = (n + 127) / 128;
  a.inv_sqrt_m = static_cast<float>(1.0 / std::sqrt(static_cast<double>(m)));
  a.log2_m = -0.5 * std::log2(static_cast<double>(m));
  if (trf) return bf16 ? go<uint16_t, true>(a, st) : go<float, true>(a, st);
  return bf16 ? go<uint16_t, false>(a, st) : go<float, false>(a, st);
}

}  // namespace krpe
