// The Toeplitz product alone (krpe_toeplitz_conv) for n <= 8192: one kernel
// per call after the spectrum of c.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "common.hpp"
#include "launch.hpp"

namespace krpe {

// Transform of the kernel: the forward's, with twiddle tables in thread order
// up to N = 4096 (at 8192, 512 threads, the compact tables).
template <int L2>
struct ToepFft {
  using C = Conf<L2>;
  static constexpr bool TWT = L2 <= 12;  // (toeplitz_tables)
  using F = Fft<C::L2T, C::LOG2R, 1 + L2 - C::L2T, C::TWC, false, C::PAD, TWT>;
  static constexpr int TABLE = TWT ? (F::P - 1) * F::N : 0;  // entries of the thread-order tables
  static_assert(TABLE <= 2 * F::N, "thread-order tables: at most 2 N entries");
};

// W_{2N} and the thread-order tables: entry (p, e, tau), e = u RP + s, is
// W_{L_p}^{t s}, t = (tau + T u) mod (L_p / RP).
template <int L2>
__global__ void k_thread_twiddles(float2* __restrict__ tw, float2* __restrict__ tt) {
  using F = typename ToepFft<L2>::F;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < 2 * F::N) {
    double sn, cs;
    sincospi(-static_cast<double>(i) / static_cast<double>(F::N), &sn, &cs);
    tw[i] = make_float2(static_cast<float>(cs), static_cast<float>(sn));
  } else if (i < 2 * F::N + ToepFft<L2>::TABLE) {
    const int j = i - 2 * F::N, p = j / F::N, e = (j % F::N) / F::T, tau = j % F::T;
    const int lrp = F::lr(p), rp = 1 << lrp, len = F::N >> (F::LR * p), sp = len >> lrp;
    const int u = e / rp, s = e % rp, t = (tau + F::T * u) % sp;
    double sn, cs;
    sincospi(-2.0 * static_cast<double>(t * s % len) / static_cast<double>(len), &sn, &cs);
    tt[j] = make_float2(static_cast<float>(cs), static_cast<float>(sn));
  }
}

// y = C a for a pair of channels of one (batch, head) per unit: both channels
// are read once into registers, brought to the power of two of their largest
// entries and packed as one complex signal (as the forward pass packs value
// columns), run through both residue classes of the length-2N transform, and
// written once.  Through the forward's convolution kernel (one feature equal
// to 1) the channels were read for their maxima, read and written packed, read
// once per class, and the classes' partial sums written, read and added.  At
// 96 heads, 64 channels, n = 4096: 345 -> 131 us per call, 115 this kernel.
// The channels once in and out are 0.2 GB, 42 us at a plain copy's rate, the
// transforms about 50 us of the VALU; the rest is the latency of each unit's
// serial chain at two work-groups per CU.  Measured and not kept: twiddles and
// twists kept over the classes (they spill, 209 us), twiddles gathered from
// W_{2N} (224), the channels re-read per class at two or three work-groups per
// CU (171 and 187 us per call).
template <int L2>
__global__ __launch_bounds__(Conf<L2>::THREADS) __attribute__((amdgpu_waves_per_eu(2))) void k_toeplitz(
    const float* __restrict__ a, const float2* __restrict__ Hs, const float2* __restrict__ tw, const float2* __restrict__ tt,
    float* __restrict__ y, int H, int n, int C, int units) {
  using Cf = Conf<L2>;
  using F = typename ToepFft<L2>::F;
  static_assert(Cf::FOLD == 1, "k_toeplitz: one transform per class");
  constexpr int S = Cf::S;
  __shared__ float2 lds_all[Cf::LDS_SLOTS];
  __shared__ float red[Cf::WAVES];
  const int g = Cf::G == 1 ? 0 : threadIdx.x / F::T, tau = Cf::G == 1 ? threadIdx.x : threadIdx.x % F::T;
  const int pairs = (C + 1) / 2;
  int unit = xcd_block(blockIdx.x, gridDim.x) * Cf::G + g;
  const bool active = unit < units;
  if (!active) unit = units - 1;  // keeps the barriers uniform, results discarded
  const int cp = unit % pairs, bh = unit / pairs, h = bh % H;
  const int c0 = 2 * cp;
  const bool two = c0 + 1 < C;
  float2* lds = lds_all + g * (F::P > 1 ? F::LDS : 0);
  const float* __restrict__ a0 = a + (static_cast<size_t>(bh) * C + c0) * n;
  const float* __restrict__ a1 = two ? a0 + n : a0;
  float2 v[F::R];
#pragma unroll
  for (int i = 0; i < F::R; ++i) {
    const int pos = tau + F::T * i, at = min(pos, n - 1);
    v[i] = make_float2(a0[at], a1[at]);
    if (pos >= n) v[i].x = 0.f;
    if (pos >= n || !two) v[i].y = 0.f;
  }
  float m0 = 0.f, m1 = 0.f;
#pragma unroll
  for (int i = 0; i < F::R; ++i) {
    m0 = fmaxf(m0, fabsf(v[i].x));
    m1 = fmaxf(m1, fabsf(v[i].y));
  }
  const float s0 = unit_reduce<F::T>(m0, red, OpMax()), s1 = unit_reduce<F::T>(m1, red, OpMax());
  // the power of two of each channel's largest entry
  const int e0 = __builtin_amdgcn_frexp_expf(s0), e1 = __builtin_amdgcn_frexp_expf(s1);
#pragma unroll
  for (int i = 0; i < F::R; ++i) v[i] = make_float2(ldexpf(v[i].x, -e0), ldexpf(v[i].y, -e1));
  float2 acc[F::R];
  constexpr_for<S>([&](auto rc) {
    constexpr int r = decltype(rc)::value;
    // the twiddles and twists are re-read in each transform: kept, they cost
    // the registers of a work-group per CU
    const float2* __restrict__ tf = tt;
    const float2* __restrict__ ti = tt;
    const float2* __restrict__ wf = tw;
    const float2* __restrict__ wi = tw;
    asm volatile("" : "+s"(tf));
    asm volatile("" : "+s"(ti));
    asm volatile("" : "+s"(wf));
    asm volatile("" : "+s"(wi));
    float2 x[F::R];
#pragma unroll
    for (int i = 0; i < F::R; ++i) x[i] = r == 0 ? v[i] : cmul(v[i], wf[r * (tau + F::T * i)]);
    if constexpr (r > 0 && F::P > 1) __syncthreads();  // the previous class's last reads
    F::forward(x, lds, tf, tau);
    const float2* __restrict__ Hh = Hs + (static_cast<size_t>(h) * S + r) * F::N;
#pragma unroll
    for (int i = 0; i < F::R; ++i) x[i] = cmul(x[i], Hh[i * F::T + tau]);
    F::inverse(x, lds, ti, tau);
#pragma unroll
    for (int i = 0; i < F::R; ++i) {
      const float2 t = r == 0 ? x[i] : cmulc(x[i], wi[r * (tau + F::T * i)]);
      acc[i] = r == 0 ? t : cadd(acc[i], t);
    }
  });
  if (!active) return;
  float* __restrict__ y0 = y + (static_cast<size_t>(bh) * C + c0) * n;
#pragma unroll
  for (int i = 0; i < F::R; ++i) {
    const int pos = tau + F::T * i;
    if (pos < n) {
      y0[pos] = ldexpf(acc[i].x, e0);
      if (two) y0[n + pos] = ldexpf(acc[i].y, e1);
    }
  }
}

namespace {

template <int L2 = 0>
hipError_t go(int l2, const float* a, const float2* Hs, const float2* tw, const float2* tt, float* y, int BH, int H, int n, int C,
              hipStream_t st) {
  if constexpr (L2 > kToeplitzLog2N) {
    return hipErrorInvalidValue;
  } else {
    if (l2 != L2) return go<L2 + 1>(l2, a, Hs, tw, tt, y, BH, H, n, C, st);
    using Cf = Conf<L2>;
    const long long units = static_cast<long long>(BH) * ((C + 1) / 2);
    const long long blocks = (units + Cf::G - 1) / Cf::G;
    hipLaunchKernelGGL(k_toeplitz<L2>, dim3(static_cast<unsigned>(blocks)), dim3(Cf::THREADS), 0, st, a, Hs, tw, tt, y, H, n,
                       C, static_cast<int>(units));
    return hipGetLastError();
  }
}

}  // namespace

namespace {
template <int L2 = 0>
hipError_t go_twiddles(int l2, float2* tw, float2* tt, hipStream_t st) {
  if constexpr (L2 > kToeplitzLog2N) {
    return hipErrorInvalidValue;
  } else {
    if (l2 != L2) return go_twiddles<L2 + 1>(l2, tw, tt, st);
    if constexpr (!ToepFft<L2>::TWT) {
      return launch_twiddles(tw, L2, st);
    } else {
      const int count = (2 << L2) + ToepFft<L2>::TABLE;
      hipLaunchKernelGGL(k_thread_twiddles<L2>, dim3((count + 255) / 256), dim3(256), 0, st, tw, tt);
      return hipGetLastError();
    }
  }
}
}  // namespace

bool toeplitz_tables(int l2) { return l2 <= 12; }

hipError_t launch_toeplitz_twiddles(int l2, float2* tw, float2* tt, hipStream_t st) { return go_twiddles(l2, tw, tt, st); }

hipError_t launch_toeplitz(int l2, const float* a, const float2* Hs, const float2* tw, const float2* tt, float* y, int BH,
                           int H, int n, int C, hipStream_t st) {
  return go(l2, a, Hs, tw, toeplitz_tables(l2) ? tt : tw, y, BH, H, n, C, st);
}

}  // namespace krpe
