// The direct route: Eq. (10) evaluated as (phi(Q) phi(K)^T o C) [v, 1] on the
// fp16 matrix cores at fp32 accuracy (wprod.hpp), two launches (three where
// the keys of a row tile are split over work-groups):
//
//  k_prep          phi(q), phi(k) and v as fragments, the table of c = exp(b).
//  k_direct        the two products of 128 rows over their keys.
//  k_direct_parts  sums the parts of a split row tile.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"
#include "direct_kernel.hpp"
#include "wprod.hpp"

namespace krpe {

// ----------------------------------------------------------------- prep --
// One launch, three kinds of work-group (by block index):
//  phi  128 positions of one (source, batch-head): the projections s = W x on
//       the bf16 matrix cores (operands in three bf16 terms, split in
//       registers and LDS; six products, three for bf16 x), the feature map
//       of Sec. 2 on the accumulators, and the result, scaled by the power of
//       two of the position's largest feature, as S fragments, whose lane
//       order is the accumulators'.  Features of the trigonometric map: sines
//       in k steps [0, KS / 2), cosines in the rest (the contraction does not
//       see their order; unused slots are zero, as are positions >= n).
//  v    128 positions of one batch-head as Z fragments.  An element that is
//       not finite is stored as zero and its block flagged: k_direct adds
//       its contribution separately (a split of it would give inf - inf),
//       as it does elements 2^31 (bf16: 2^32) and more below their
//       block's largest, whose power they share.
//  c    2048 entries of one head's table and the range of its finite ones.
// The features are written once and read once per 128 rows; at 96 heads, n =
// 4096, m = 128 the kernel is bound by its 0.5 GB of stores.
struct PrepArgs {
  const void *q, *k, *v;
  const float *W, *b;
  uint4 *X, *Y, *Z;
  float* krec;      // [BH][nblk][64] (KeyRec)
  unsigned* vflag;  // [BH][nblk]
  float* ctab;      // [H][ctab_stride]
  int2* crange;     // [H][ctab_chunks]
  float* crev;      // the table and ranges of c_{-t} (NULL: not wanted)
  int2* rrange;
  unsigned* fix;    // fix[BH] = rows evaluated exactly (all of them)
  int *qpow, *kpow; // [BH][32 nblk] powers of phi(q), phi(k) (kpow NULL: not wanted)
  float* qsum;      // [BH][32 nblk] sums of phi(q) in units of its power
  unsigned* flag;   // [BH + 1] cleared
  int BH, H, n, nblk, d, m, KS, ct_total, kind, nprf, tiles, phi_blocks, v_blocks;
  float inv_sqrt_m;
  double log2_m;  // -log2(sqrt(m))
};
// DK: k steps of the head dimension, d <= 16 DK.  NT: 32-feature tiles of
// projections held in registers until the position's largest feature is known.
template <typename TX, int DK, int NT>
__device__ __forceinline__ void prep_phi(const PrepArgs& a, int bid, float* __restrict__ smem) {
  constexpr int XS = x_stride(DK);
  constexpr int NSX = sizeof(TX) == 2 ? 1 : 3;
  constexpr int GT = DK <= 4 ? 4 : 2;  // tiles of W staged at a time
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 31, lh = lane >> 5;
  const int pt = bid % a.tiles, rest = bid / a.tiles, bh = rest % a.BH, src = rest / a.BH;
  const int h = bh % a.H, n = a.n, d = a.d;
  const TX* __restrict__ x = static_cast<const TX*>(src == 0 ? a.q : a.k) + static_cast<size_t>(bh) * n * d;
  const int p0 = pt * 128, rows = min(128, n - p0);
  __shared__ int wodd;
  if (tid == 0) wodd = 0;
  stage_x<TX, DK>(x, p0, rows, d, smem);
  __syncthreads();
  // this lane's position: its operand and squared norm
  uint4 xf[DK][NSX];
  const float* __restrict__ row = smem + (32 * wave + lr) * XS;
  const double sqd = x_operand<DK, NSX>(row, lh, xf);
  const bool xodd = __any(unsplit(sqd));  // uniform
  bool plain = xodd;
  // phi of x / ||x|| when normalising (Algorithm 1, first step): the
  // projections scale by 1 / ||x|| and ||x||^2 / 2 becomes 1/2 (a zero row
  // stays zero).
  const bool nz = sqd > 0.0;
  const double half_sq = a.nprf ? (nz ? 0.5 : 0.0) : 0.5 * sqd;
  const float row_scale = a.nprf ? (nz ? static_cast<float>(1.0 / sqrt(sqd)) : 0.f) : 1.f;
  // PRF: phi_prf's factors
  const float rs = static_cast<float>((a.nprf ? (nz ? 1.0 / sqrt(sqd) : 0.0) : 1.0) * kLog2e);
  const double e0d = a.log2_m - half_sq * kLog2e;
  const float e0 = static_cast<float>(e0d), ef = rounding_factor(e0d, e0);
  const bool pos_ok = p0 + 32 * wave + lr < n;
  const int blk = 4 * pt + wave;
  const bool store = blk < a.nblk;  // uniform
  const size_t block = static_cast<size_t>(bh) * a.nblk + min(blk, a.nblk - 1);
  uint4* __restrict__ ob = (src == 0 ? a.X : a.Y) + block * a.KS * 2 * kFragLanes + lane;
  const int ksp = a.kind == kFeatTrf ? a.KS / 2 : a.KS;  // k steps of projections (of x for elu + 1)
  const int ftiles = (ksp + 1) / 2;
  const float* __restrict__ Wh = a.W + static_cast<size_t>(h) * a.m * d;
  uint4* __restrict__ wf = reinterpret_cast<uint4*>(smem);
  auto stage_tiles = [&](int t0) {
    __syncthreads();  // x rows / the previous features consumed
    stage_w<DK>(Wh, 32 * t0, min(GT, ftiles - t0), a.m, d, wf, &wodd);
    __syncthreads();
    plain = xodd || __builtin_amdgcn_readfirstlane(wodd) != 0;
  };
  auto project_tile = [&](int ti, int t0, floatx16& acc, floatx16& lo) {
    project<DK, NSX, false>(wf + (ti - t0) * DK * 3 * kFragLanes, xf, acc, lo);
    if (__builtin_expect(plain, 0)) {
      project_plain(Wh + static_cast<size_t>(min(32 * ti + lr, a.m - 1)) * d,
                    x + static_cast<size_t>(min(p0 + 32 * wave + lr, n - 1)) * d, d, acc);
      lo = zero16();
    }
  };
  auto emit = [&](int ks, const float (&v8)[8]) {
    uint4 hh, ll;
    split_f16x8(v8, kLoScale, hh, ll);
    ob[(ks * 2 + 0) * kFragLanes] = hh;
    ob[(ks * 2 + 1) * kFragLanes] = ll;
  };
  int ex;  // the position's power: its largest feature is brought to [2^14, 2^15)
  bool any_phi;
  float sum = 0.f;
  if (a.kind == kFeatTrf) {
    // every feature is at most the amplitude: no need to see them first
    const float amp = pos_ok ? static_cast<float>(exp(half_sq)) * a.inv_sqrt_m : 0.f;
    ex = __builtin_amdgcn_frexp_expf(amp) - 15;
    const float as = ldexpf(amp, -ex);
    any_phi = amp > 0.f;
    for (int t0 = 0; t0 < ftiles; t0 += GT) {
      stage_tiles(t0);
      for (int tt = 0; tt < min(GT, ftiles - t0) && store; ++tt) {
        floatx16 acc, lo;
        project_tile(t0 + tt, t0, acc, lo);
        float s16[16], c16[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const bool in = 32 * (t0 + tt) + 8 * (e >> 2) + 4 * lh + (e & 3) < a.m;
          sincosf((acc[e] + lo[e]) * row_scale, &s16[e], &c16[e]);
          s16[e] = in ? s16[e] * as : 0.f;
          c16[e] = in ? c16[e] * as : 0.f;
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int ks = 2 * (t0 + tt) + j;
          if (ks >= ksp) continue;  // uniform
          float v8[8];
#pragma unroll
          for (int t = 0; t < 8; ++t) v8[t] = s16[8 * j + t];
          emit(ks, v8);
#pragma unroll
          for (int t = 0; t < 8; ++t) v8[t] = c16[8 * j + t];
          emit(ksp + ks, v8);
        }
      }
    }
  } else {
    float val[NT][16];
    if (a.kind == kFeatElu) {
      constexpr_for<NT>([&](auto tc) {
        constexpr int t0 = decltype(tc)::value;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          // x_f + 1 for x_f > 0, exp(x_f) otherwise
          const int f = 32 * t0 + 8 * (e >> 2) + 4 * lh + (e & 3);
          const float y = f < d ? row[f] * row_scale : 0.f;
          val[t0][e] = f < d && pos_ok ? (y > 0.f ? y + 1.f : expf(y)) : 0.f;
        }
      });
    } else {
      constexpr_for<NT>([&](auto tc) {
        constexpr int ti = decltype(tc)::value, t0 = ti / GT * GT;
        if (ti >= ftiles) return;  // uniform
        if constexpr (ti == t0) stage_tiles(t0);
        floatx16 acc, lo;
        project_tile(ti, t0, acc, lo);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          val[ti][e] = pos_ok ? phi_prf(acc[e], lo[e], rs, e0, ef) : 0.f;
        }
        if (32 * ti + 32 > a.m) {  // uniform: unused slots are zero
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if (32 * ti + 8 * (e >> 2) + 4 * lh + (e & 3) >= a.m) val[ti][e] = 0.f;
        }
      });
    }
    float mx = 0.f;
    constexpr_for<NT>([&](auto tc) {
      constexpr int ti = decltype(tc)::value;
      if (ti < ftiles) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          mx = fmaxf(mx, val[ti][e]);
          sum += val[ti][e];
        }
      }
    });
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    sum += __shfl_xor(sum, 32);
    ex = __builtin_amdgcn_frexp_expf(mx) - 15;  // (-15 for zero, infinite and NaN maxima)
    any_phi = mx > 0.f;
    constexpr_for<2 * NT>([&](auto kc) {
      constexpr int ks = decltype(kc)::value;
      if (ks >= ksp || !store) return;  // uniform
      float v8[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) v8[t] = ldexpf(val[ks / 2][8 * (ks % 2) + t], -ex);
      emit(ks, v8);
    });
  }
  if (src == 0 && pt == 0 && tid == 0) a.flag[bh] = 0u;
  if (!store) return;
  sum = ldexpf(sum, -ex);
  if (src == 0) {
    if (lh == 0) {
      a.qpow[block * kBlk + lr] = ex;
      a.qsum[block * kBlk + lr] = sum;
    }
  } else {
    if (a.kpow && lh == 0) a.kpow[block * kBlk + lr] = ex;
    // (positions without features have no power of their own)
    int E = any_phi ? ex : -400;
#pragma unroll
    for (int off = 16; off > 0; off >>= 1) {
      E = max(E, __shfl_xor(E, off));
      sum = fmaxf(sum, __shfl_xor(sum, off));
    }
    float* __restrict__ rec = a.krec + block * kRecWords;
    if (lh == 0) rec[lr] = any_phi ? ldexpf(1.f, ex - E - kRecBias) : 0.f;
    if (lane == 0) {
      rec[kRecE] = __int_as_float(E + kRecBias);
      rec[kRecSum] = sum;
    }
  }
}

template <typename TX>
__device__ __forceinline__ void prep_v(const PrepArgs& a, int bid) {
  // (bf16 values: 8 significant bits, one fp16 term holds them)
  constexpr int NSZ = sizeof(TX) == 2 ? 1 : 2;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 31, lh = lane >> 5, n = a.n, d = a.d;
  const int pt = bid % a.tiles, bh = bid / a.tiles, blk = 4 * pt + wave;
  if (blk >= a.nblk) return;  // uniform per wave; no barrier in this role
  const TX* __restrict__ v = static_cast<const TX*>(a.v) + static_cast<size_t>(bh) * n * d;
  const size_t block = static_cast<size_t>(bh) * a.nblk + blk;
  uint4* __restrict__ out = a.Z + block * a.ct_total * 2 * NSZ * kFragLanes + lane;
  bool odd = false, lost = false;
  float x[kMaxD / 32][16];
  float mx = 0.f;
#pragma unroll
  for (int ct = 0; ct < kMaxD / 32; ++ct) {
    if (ct >= a.ct_total) continue;  // uniform
    const int col = 32 * ct + lr;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int pos = 32 * blk + 8 * (e >> 2) + 4 * lh + (e & 3);
      x[ct][e] = pos < n && col < d ? to_f32(v[static_cast<size_t>(pos) * d + col]) : 0.f;
    }
  }
#pragma unroll
  for (int ct = 0; ct < kMaxD / 32; ++ct) {
    if (ct >= a.ct_total) continue;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      if (!isfinite(x[ct][e])) {
        x[ct][e] = 0.f;
        odd = true;
      }
      mx = fmaxf(mx, fabsf(x[ct][e]));
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
  const int ex = __builtin_amdgcn_frexp_expf(mx) - 15;
#pragma unroll
  for (int ct = 0; ct < kMaxD / 32; ++ct) {
    if (ct >= a.ct_total) continue;
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2) {
      float v8[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        v8[t] = ldexpf(x[ct][8 * k2 + t], -ex);
        const float small = apart<NSZ>(v8[t]);
        lost |= small != 0.f;
        v8[t] -= small;
      }
      uint4 hh, ll;
      split_f16x8(v8, kLoScale, hh, ll);
      out[((ct * 2 + k2) * NSZ + 0) * kFragLanes] = hh;
      if (NSZ > 1) out[((ct * 2 + k2) * NSZ + NSZ - 1) * kFragLanes] = ll;
    }
  }
  const unsigned any = (__any(odd) ? 1u : 0u) | (__any(lost) ? 2u : 0u);
  if (lane == 0) {
    a.vflag[block] = any;
    a.krec[block * kRecWords + kRecV] = __int_as_float(ex);
  }
}

__device__ __forceinline__ void prep_c(const PrepArgs& a, int bid) {
  __shared__ int2 wr[4];
  const int chunks = ctab_chunks(a.n), stride = ctab_stride(a.n), len = 2 * a.n - 1;
  const int h = bid / chunks, ch = bid % chunks;
  const float* __restrict__ bh = a.b + static_cast<size_t>(h) * len;
  float* __restrict__ ct = a.ctab + static_cast<size_t>(h) * stride;
  int lo = 1 << 30, hi = -1;
  float v[kCChunk / 256];
#pragma unroll
  for (int j = 0; j < kCChunk / 256; ++j) {
    const int s = ch * kCChunk + 256 * j + static_cast<int>(threadIdx.x) - kCPad;
    v[j] = s >= 0 && s < len ? bh[s] : -INFINITY;
  }
#pragma unroll
  for (int j = 0; j < kCChunk / 256; ++j) {
    const int e = ch * kCChunk + 256 * j + static_cast<int>(threadIdx.x), s = e - kCPad;
    const float cv = s >= 0 && s < len ? expf(v[j]) : 0.f;
    if (e < stride) ct[e] = cv;
    if (a.crev && e < stride) {
      // (the pads of the reversed table are written by the entries past len)
      float* __restrict__ cr = a.crev + static_cast<size_t>(h) * stride;
      if (s >= 0 && s < len) {
        cr[kCPad + len - 1 - s] = cv;
      } else {
        cr[e] = 0.f;
      }
    }
    if (s >= 0 && s < len && v[j] != -INFINITY) {
      lo = min(lo, s);
      hi = max(hi, s);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    lo = min(lo, __shfl_xor(lo, off));
    hi = max(hi, __shfl_xor(hi, off));
  }
  if ((threadIdx.x & 63) == 0) wr[threadIdx.x >> 6] = make_int2(lo, hi);
  __syncthreads();
  if (threadIdx.x == 0) {
    lo = min(min(wr[0].x, wr[1].x), min(wr[2].x, wr[3].x));
    hi = max(max(wr[0].y, wr[1].y), max(wr[2].y, wr[3].y));
    a.crange[static_cast<size_t>(h) * chunks + ch] = make_int2(lo, hi);
    if (a.crev) a.rrange[static_cast<size_t>(h) * chunks + ch] = hi < 0 ? make_int2(lo, hi) : make_int2(len - 1 - hi, len - 1 - lo);
    if (bid == 0) {
      a.fix[a.BH] = static_cast<unsigned>(a.BH) * static_cast<unsigned>(a.n);
      a.flag[a.BH] = 0u;
    }
  }
}

template <typename TX, int DK, int NT>
__global__ __launch_bounds__(256) void k_prep(PrepArgs a) {
  constexpr int kX = 128 * x_stride(DK), kW = (DK <= 4 ? 4 : 2) * DK * 3 * 256;
  __shared__ __align__(16) float smem[kX > kW ? kX : kW];
  const int bid = blockIdx.x;
  if (bid < a.phi_blocks) {
    prep_phi<TX, DK, NT>(a, bid, smem);
  } else if (bid < a.phi_blocks + a.v_blocks) {
    prep_v<TX>(a, bid - a.phi_blocks);
  } else {
    prep_c(a, bid - a.phi_blocks - a.v_blocks);
  }
}

// z of a split row tile: its parts' numerators and denominators summed in
// part order.  Work-group: the tile's rows and 8 of its columns (lanes along
// the rows, the order of the parts in memory).
template <int CT, int NW>
__global__ __launch_bounds__(64 * NW) void k_direct_parts(DirectArgs a) {
  constexpr int cw = CT * 32 + 1, kRows = 32 * NW;
  const int row = threadIdx.x % kRows, cg = threadIdx.x / kRows;
  int b = blockIdx.x;
  const int grp = b % (CT * 4);
  b /= CT * 4;
  const int tile = b % a.tiles;
  b /= a.tiles;
  const int pass = b % a.passes, bh = b / a.passes, i = tile * kRows + row;
  const int cl = 8 * grp + 4 * cg, c = pass * CT * 32 + cl;
  if (i >= a.n || c >= a.d) return;
  const double* __restrict__ part =
      a.part + (static_cast<size_t>(bh * a.passes + pass) * a.tiles + tile) * a.nparts * (kRows * cw) + row;
  double num[4] = {0.0, 0.0, 0.0, 0.0}, den = 0.0;
  for (int p = 0; p < a.nparts; ++p) {
    const double* __restrict__ q = part + static_cast<size_t>(p) * (kRows * cw);
#pragma unroll
    for (int j = 0; j < 4; ++j) num[j] += q[(cl + j) * kRows];
    den += q[CT * 32 * kRows];
  }
  float* __restrict__ zr = a.z + (static_cast<size_t>(bh) * a.n + i) * a.d;
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (c + j < a.d) zr[c + j] = static_cast<float>(num[j] / den);
  if (c == 0 && a.den) a.den[static_cast<size_t>(bh) * a.n + i] = den;
}

// ------------------------------------------------------------ launchers --
namespace {

float inv_sqrt(int m) { return static_cast<float>(1.0 / std::sqrt(static_cast<double>(m))); }
double log2_scale(int m) { return -0.5 * std::log2(static_cast<double>(m)); }  // -log2(sqrt(m))

// k steps the kernels are compiled for
int round_ks(int ks) {
  for (int k : {2, 4, 6, 8, 12, 16})
    if (ks <= k) return k;
  return 0;
}

// Waves (of 32 rows) per work-group.
constexpr int direct_waves(int KS) { return 4; }

template <int NSZ, int KS, int CT>
hipError_t direct_go(const DirectArgs& a, hipStream_t st) {
  constexpr int NW = direct_waves(KS);
  const long long blocks = static_cast<long long>(a.BH) * a.passes * a.tiles * a.nparts;
  hipLaunchKernelGGL((k_direct<0, NSZ, KS, 0, CT, NW>), dim3(static_cast<unsigned>(blocks)), dim3(64 * NW), 0, st, a);
  if (hipError_t e = hipGetLastError(); e != hipSuccess || a.nparts == 1) return e;
  hipLaunchKernelGGL((k_direct_parts<CT, NW>),
                     dim3(static_cast<unsigned>(static_cast<long long>(a.BH) * a.passes * a.tiles * (CT * 4))),
                     dim3(64 * NW), 0, st, a);
  return hipGetLastError();
}

template <int NSZ, int CT>
hipError_t direct_ks(int KS, const DirectArgs& a, hipStream_t st) {
  switch (KS) {
    case 2: return direct_go<NSZ, 2, CT>(a, st);
    case 4: return direct_go<NSZ, 4, CT>(a, st);
    case 6: return direct_go<NSZ, 6, CT>(a, st);
    case 8: return direct_go<NSZ, 8, CT>(a, st);
    case 12: return direct_go<NSZ, 12, CT>(a, st);
    case 16: return direct_go<NSZ, 16, CT>(a, st);
    default: return hipErrorInvalidValue;
  }
}

template <typename TX, int DK>
hipError_t prep_nt(const PrepArgs& a, hipStream_t st) {
  const dim3 grid(static_cast<unsigned>(a.phi_blocks + a.v_blocks + a.H * ctab_chunks(a.n)));
  const int ftiles = ((a.kind == kFeatTrf ? a.KS / 2 : a.KS) + 1) / 2;
  if (ftiles <= 2)
    hipLaunchKernelGGL((k_prep<TX, DK, 2>), grid, dim3(256), 0, st, a);
  else if (ftiles <= 4)
    hipLaunchKernelGGL((k_prep<TX, DK, 4>), grid, dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL((k_prep<TX, DK, 8>), grid, dim3(256), 0, st, a);
  return hipGetLastError();
}
template <typename TX>
hipError_t prep_go(const PrepArgs& a, hipStream_t st) {
  if (a.d <= 32) return prep_nt<TX, 2>(a, st);
  if (a.d <= 64) return prep_nt<TX, 4>(a, st);
  return prep_nt<TX, 8>(a, st);
}

}  // namespace

int direct_ksteps(int kind, int d, int m) {
  const int rows = kind == kFeatElu ? d : m;
  const int ks = (rows + 15) / 16;
  return round_ks(kind == kFeatTrf ? 2 * ks : ks);
}

// Parts a row tile's key blocks are split into.  W work-groups of nb key
// blocks each fill the chip in rounds of its resident ones (two per CU, one
// with more than 128 features); p parts cost ceil(W p / resident) rounds of
// nb / p blocks and a fixed two, plus the partial sums' round trip (33 KB of
// fp64 per 32 columns and part at about 4 TB/s, in units of a key block's
// about 1 us).
int direct_parts(long long BH, int n, int ct_total, int KS) {
  const int ct = ct_total >= 2 ? 2 : 1, passes = (ct_total + ct - 1) / ct;
  const int nb = (n + kBlk - 1) / kBlk;
  const int rows = 32 * direct_waves(KS);
  const long long W = BH * passes * ((n + rows - 1) / rows);
  const long long resident = KS <= 8 ? 512 : 256;
  if (W >= 4 * resident) return 1;
  int best = 1;
  double cost = 0.0;
  for (int p = 1; p <= 32 && (p == 1 || nb / p >= 4); ++p) {
    const double rounds = static_cast<double>((W * p + resident - 1) / resident);
    const double c = rounds * (static_cast<double>(nb) / p + 2.0) +
                     (p > 1 ? 4.0 + static_cast<double>(W) * p * ct * 33e3 * 2.0 / 4e6 : 0.0);
    if (p == 1 || c < cost) {
      best = p;
      cost = c;
    }
  }
  return best;
}

DirectLayout direct_layout(int B, int H, int n, int d, int ks) {
  DirectLayout L{};
  const size_t bh = static_cast<size_t>(B) * H;
  L.nblk = (n + kBlk - 1) / kBlk;
  L.ks = ks;
  const int ct = (d + 31) / 32;
  L.passes = (ct + 1) / 2;
  L.ct_total = ct >= 2 ? 2 * L.passes : 1;
  L.nparts = direct_parts(static_cast<long long>(bh), n, L.ct_total, ks);
  size_t off = 0;
  auto take = [&off](size_t bytes) {
    const size_t at = off;
    off = (off + bytes + 255) & ~static_cast<size_t>(255);
    return at;
  };
  constexpr size_t kFrag = kFragLanes * sizeof(uint4);
  L.fix = take((bh + 1) * sizeof(unsigned));
  L.x = take(bh * L.nblk * ks * 2 * kFrag);
  L.y = take(bh * L.nblk * ks * 2 * kFrag);
  L.z = take(bh * L.nblk * L.ct_total * 2 * 2 * kFrag);
  L.krec = take(bh * L.nblk * kRecWords * sizeof(float));
  L.vflag = take(bh * L.nblk * sizeof(unsigned));
  L.ctab = take(static_cast<size_t>(H) * ctab_stride(n) * sizeof(float));
  L.crange = take(static_cast<size_t>(H) * ctab_chunks(n) * sizeof(int2));
  L.qpow = take(bh * L.nblk * kBlk * sizeof(int));
  L.qsum = take(bh * L.nblk * kBlk * sizeof(float));
  L.flag = take((bh + 1) * sizeof(unsigned));
  const size_t rows = 32 * direct_waves(ks), tiles = (static_cast<size_t>(n) + rows - 1) / rows;
  const size_t cw = (L.ct_total >= 2 ? 64 : 32) + 1;
  L.part = take(L.nparts > 1 ? bh * L.passes * tiles * L.nparts * rows * cw * sizeof(double) : 0);
  L.total = off;
  return L;
}

hipError_t launch_direct_prep(const DirectLayout& L, char* w, const void* q, const void* k, const void* v, bool bf16,
                              const float* b, const float* W, int BH, int H, int n, int d, int m, bool nprf, int kind,
                              int* kpow, float* crev, int2* rrange, hipStream_t st) {
  PrepArgs p{};
  p.kpow = kpow, p.crev = crev, p.rrange = rrange;
  p.q = q, p.k = k, p.v = v, p.W = W, p.b = b;
  p.X = reinterpret_cast<uint4*>(w + L.x);
  p.Y = reinterpret_cast<uint4*>(w + L.y);
  p.Z = reinterpret_cast<uint4*>(w + L.z);
  p.vflag = reinterpret_cast<unsigned*>(w + L.vflag);
  p.ctab = reinterpret_cast<float*>(w + L.ctab);
  p.crange = reinterpret_cast<int2*>(w + L.crange);
  p.fix = reinterpret_cast<unsigned*>(w + L.fix);
  p.BH = BH, p.H = H, p.n = n, p.nblk = L.nblk, p.d = d, p.m = m, p.KS = L.ks, p.ct_total = L.ct_total;
  p.kind = kind, p.nprf = nprf ? 1 : 0;
  p.krec = reinterpret_cast<float*>(w + L.krec);
  p.qpow = reinterpret_cast<int*>(w + L.qpow);
  p.qsum = reinterpret_cast<float*>(w + L.qsum);
  p.flag = reinterpret_cast<unsigned*>(w + L.flag);
  p.tiles = (n + 127) / 128;
  p.phi_blocks = 2 * BH * p.tiles;
  p.v_blocks = BH * p.tiles;
  p.inv_sqrt_m = inv_sqrt(m);
  p.log2_m = log2_scale(m);
  return bf16 ? prep_go<uint16_t>(p, st) : prep_go<float>(p, st);
}

void direct_exact_args(const DirectLayout& L, char* w, const void* q, const void* k, const void* v, bool bf16,
                       const float* W, int BH, int H, int n, int d, int m, bool nprf, int kind, DirectArgs& a) {
  a.q = q, a.k = k, a.v = v, a.W = W, a.m = m, a.kind = kind, a.nprf = nprf ? 1 : 0;
  a.BH = BH, a.H = H, a.n = n, a.nblk = L.nblk, a.d = d;
  a.ctab = reinterpret_cast<const float*>(w + L.ctab);
  a.crange = reinterpret_cast<const int2*>(w + L.crange);
  a.qpow = reinterpret_cast<const int*>(w + L.qpow);
  a.qsum = reinterpret_cast<const float*>(w + L.qsum);
  a.flag = reinterpret_cast<unsigned*>(w + L.flag);
  a.inv_sqrt_m = inv_sqrt(m), a.log2_m = log2_scale(m);
}

hipError_t launch_direct(const DirectLayout& L, char* w, const void* q, const void* k, const void* v, bool bf16,
                         const float* W, float* z, double* den, int BH, int H, int n, int d, int m, bool nprf, int kind,
                         hipStream_t st) {
  DirectArgs a{};
  a.X = reinterpret_cast<const uint4*>(w + L.x);
  a.Y = reinterpret_cast<const uint4*>(w + L.y);
  a.Z = reinterpret_cast<const uint4*>(w + L.z);
  a.vflag = reinterpret_cast<const unsigned*>(w + L.vflag);
  a.z = z, a.den = den, a.part = reinterpret_cast<double*>(w + L.part);
  a.ct_total = L.ct_total;
  a.krec = reinterpret_cast<const float*>(w + L.krec);
  const int rows = 32 * direct_waves(L.ks);
  a.tiles = (n + rows - 1) / rows;
  a.passes = L.passes, a.nparts = L.nparts;
  a.remap = direct_remap(BH);
  direct_exact_args(L, w, q, k, v, bf16, W, BH, H, n, d, m, nprf, kind, a);
  if (L.ct_total >= 2)
    return bf16 ? direct_ks<1, 2>(L.ks, a, st) : direct_ks<2, 2>(L.ks, a, st);
  return bf16 ? direct_ks<1, 1>(L.ks, a, st) : direct_ks<2, 1>(L.ks, a, st);
}

}  // namespace krpe
