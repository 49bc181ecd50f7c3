// Row tiles of the direct forward pass that two fp16 terms do not hold, on the
// fp32 matrix cores: the features formed again from q, k and W, nothing split.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "common.hpp"
#include "direct_args.hpp"
#include "features.hpp"
#include "wprod.hpp"

namespace krpe {

__device__ __forceinline__ floatx16 mfma_f32(float a, float b, floatx16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// base[offset] by a 32-bit byte offset (one address register a load).
template <typename T>
__device__ __forceinline__ T at_bytes(const T* __restrict__ base, uint32_t offset) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + offset);
}

// sin x or cos x: x less its multiple of pi / 2 in fp64, then Taylor's series (up to
// r^9 and r^10, |r| <= pi / 4: below 2^-25).  sincosf takes 50 registers more.
__device__ __forceinline__ float sine(float x, bool cosine) {
  const double k = rint(static_cast<double>(x) * 0.63661977236758134);
  const float r = static_cast<float>(fma(k, -1.5707963267948966, static_cast<double>(x))), r2 = r * r;
  const int quarter = static_cast<int>(static_cast<long long>(k) & 3) + (cosine ? 1 : 0);
  const float s = fmaf(r * r2, fmaf(r2, fmaf(r2, fmaf(r2, 2.7557319e-6f, -1.9841270e-4f), 8.3333333e-3f), -0.16666667f), r);
  const float c = fmaf(
      r2, fmaf(r2, fmaf(r2, fmaf(r2, fmaf(r2, -2.7557319e-7f, 2.4801587e-5f), -1.3888889e-3f), 4.1666667e-2f), -0.5f), 1.f);
  const float y = (quarter & 1) != 0 ? c : s;
  return (quarter & 2) != 0 ? -y : y;
}

// Features of a lane's position (row xr of x, d values; `ok` false: zeros) over
// 2^pw: tile ti of 32 projections (of 32 elements of x for elu + 1), register e
// feature 32 ti + 8 (e / 4) + 4 lh + e % 4, the order of the accumulators, so
// that registers 0 .. 7 and 8 .. 15 are k steps 2 ti and 2 ti + 1 of an S
// operand.  Trigonometric map: sines, or cosines with `cosines`.
template <typename TX>
__device__ __forceinline__ void exact_features(const DirectArgs& a, const TX* __restrict__ xr, bool ok,
                                               const float* __restrict__ Wh, int ti, bool cosines, int pw,
                                               float (&out)[16]) {
  const int lane = threadIdx.x & 63, lr = lane & 31, lh = lane >> 5, d = a.d, f0 = 32 * ti;
  const bool vx = d % 8 == 0, vw = d % 4 == 0;
  const bool proj = a.kind != kFeatElu;
  const float* __restrict__ wr = proj ? Wh + static_cast<size_t>(min(f0 + lr, a.m - 1)) * d : nullptr;
  floatx16 acc = zero16();
  double sq = 0.0;
#pragma unroll 1
  for (int c = 0; c < d; c += 16) {
    const int c8 = c + 8 * lh;
    float xv[8], wv[8];
    load8(xr + c8, d - c8, vx, xv);
#pragma unroll
    for (int t = 0; t < 8; ++t) sq = fma(static_cast<double>(xv[t]), static_cast<double>(xv[t]), sq);
    if (proj) {
      load8(wr + c8, f0 + lr < a.m ? d - c8 : 0, vw, wv);
      floatx16 sum = zero16();
#pragma unroll
      for (int t = 0; t < 8; ++t) sum = mfma_f32(wv[t], xv[t], sum);
      acc += sum;  // (sums of 16 dimensions: few roundings of the whole)
    }
  }
  sq += __shfl_xor(sq, 32);
  const bool nz = sq > 0.0;
  const double half_sq = a.nprf ? (nz ? 0.5 : 0.0) : 0.5 * sq;
  const double scale = a.nprf ? (nz ? 1.0 / sqrt(sq) : 0.0) : 1.0;
  const int rows = proj ? a.m : d;
  if (a.kind == kFeatTrf) {
    const float amp = ldexpf(static_cast<float>(exp(half_sq)) * a.inv_sqrt_m, -pw);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int f = f0 + 8 * (e >> 2) + 4 * lh + (e & 3);
      const float y = sine(acc[e] * static_cast<float>(scale), cosines) * amp;
      out[e] = ok && f < rows ? y : 0.f;
      __builtin_amdgcn_sched_barrier(0);  // (few registers)
    }
    return;
  }
  const float rs = static_cast<float>(proj ? scale * kLog2e : scale);
  const double e0d = a.log2_m - half_sq * kLog2e - pw;
  const float e0 = static_cast<float>(e0d), ef = rounding_factor(e0d, e0);
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int f = f0 + 8 * (e >> 2) + 4 * lh + (e & 3);
    float y;
    if (proj) {
      y = phi_prf(acc[e], 0.f, rs, e0, ef);
    } else {
      const float x1 = f < d ? to_f32(xr[f]) * rs : 0.f;
      y = ldexpf(x1 > 0.f ? x1 + 1.f : expf(x1), -pw);
    }
    out[e] = ok && f < rows ? y : 0.f;
  }
}

// Key blocks [lo, hi) of rows r0 .. r1 under the head's range of finite b.
__device__ __forceinline__ void key_blocks(int2 br, int n, int r0, int r1, int& lo, int& hi) {
  const int jlo = max(0, r0 + br.x - (n - 1)), jhi = min(n - 1, r1 + br.y - (n - 1));
  lo = jhi >= jlo ? jlo >> 5 : 0;
  hi = jhi >= jlo ? (jhi >> 5) + 1 : 0;
}
// Columns c .. c + 3 of a row of d (16-byte aligned rows when d is a multiple of 4).
__device__ __forceinline__ void store4(float* __restrict__ row, int c, int d, float x, float y, float z, float w) {
  if (d % 4 == 0) {
    if (c < d) *reinterpret_cast<float4*>(row + c) = make_float4(x, y, z, w);
  } else {
    if (c < d) row[c] = x;
    if (c + 1 < d) row[c + 1] = y;
    if (c + 2 < d) row[c + 2] = z;
    if (c + 3 < d) row[c + 3] = w;
  }
}


// Whether every one of the 32 rows from wrow0 on passes kRowTau's test over the key
// blocks [lo, hi), given its denominator, its largest numerator, the sum of its
// weights and what it may have lost beside them (each lane its row's), first by
// the sums of the features, then in full (S formed again from memory).
template <int KS>
__device__ __forceinline__ bool rows_held(const DirectArgs& a, int bh, int wrow0, int lo, int hi, double dsum,
                                          double num, double wsum, double beside, int vmost) {
  const int lane = threadIdx.x & 63, lr = lane & 31, lh = lane >> 5, n = a.n, i = wrow0 + lr;
  const size_t hb = static_cast<size_t>(bh) * a.nblk;
  const uint4* __restrict__ xp = a.X + (hb + (wrow0 >> 5)) * KS * 2 * kFragLanes + lane;
  const float* __restrict__ ct = a.ctab + static_cast<size_t>(bh % a.H) * ctab_stride(n);
  const bool trf = a.kind == kFeatTrf;
  const double xs = trf ? 0.0 : a.qsum[(hb + (wrow0 >> 5)) * kBlk + lr];
  if (!trf) {
    float ys = 0.f;
    for (int blk = lo + lane; blk < hi; blk += 64) ys = fmaxf(ys, a.krec[(hb + blk) * kRecWords + kRecSum]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) ys = fmaxf(ys, __shfl_xor(ys, off));
    const double off = fma(kTermErr * (xs + ys), wsum, beside);
    const bool held = off <= kRowTau * dsum && fma(kSplitFloor, dsum, off) * exp2_int(vmost + 15) <= kRowTau * num;
    if (!__any(i < n && !held)) return true;
  }
  double dd = 0.0, dn = 0.0;
#pragma unroll 1
  for (int blk = lo; blk < hi; ++blk) {
    const uint4* __restrict__ yp = a.Y + (hb + blk) * KS * 2 * kFragLanes + lane;
    floatx16 s = zero16(), s1 = zero16();
#pragma unroll 1
    for (int f = 0; f < 2 * KS * kFragLanes; f += 2 * kFragLanes) {
      const uint4 xh = xp[f], xl = xp[f + kFragLanes], yh = yp[f], yl = yp[f + kFragLanes];
      s = mfma_f16(yh, xh, s);
      s1 = mfma_f16(yh, xl, s1);
      s1 = mfma_f16(yl, xh, s1);
    }
    const float* __restrict__ rec = a.krec + (hb + blk) * kRecWords;
    const int kexp = __float_as_int(rec[kRecE]), vexp = __float_as_int(rec[kRecV]);
    const double err = trf ? 0.0 : kTermErr * (xs + rec[kRecSum]);
    const float doubt = static_cast<float>(kDoubt * err);
    double w = 0.0, most = 0.0;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      if (e % 4 == 0) __builtin_amdgcn_sched_barrier(0);  // (few registers)
      const int key = 8 * (e >> 2) + 4 * lh + (e & 3), j = 32 * blk + key;
      const double c = j < n ? at_bytes(ct, static_cast<uint32_t>(j - i + kCPad + n - 1) * 4u) : 0.f;
      const double r = rec[key];
      const float se = fmaf(s1[e], kLoInv, s[e]);
      if (se < doubt) w = fma(err, r * c, w);
      // (a key of a power so far below its block's that its record is zero: at
      // most 2^38 2^-149)
      w += (r == 0.0 ? c : c > 0.0 ? 1.0 : 0.0) * kUnderflow;
      most = fmax(most, fabs(se * r * c));
    }
    dd = fma(w, exp2_int(kexp), dd);
    dn = fma(w + most * kSplitFloor, exp2_int(kexp + vexp + 15), dn);
  }
  dd += __shfl_xor(dd, 32);
  dn += __shfl_xor(dn, 32);
  // (a sum that is not finite is not held)
  return !__any(i < n && !(isfinite(dsum) && dd <= kRowTau * fabs(dsum) && dn <= kRowTau * num));
}

// Partial sums of part pi of a split row tile: [columns of the pass + 1][rows].
template <int CT, int NW>
__device__ __forceinline__ double* part_of(const DirectArgs& a, int bh, int pass, int tile, int pi) {
  constexpr int cw = CT * 32 + 1, rows = 32 * NW;
  return a.part + ((static_cast<size_t>(bh * a.passes + pass) * a.tiles + tile) * a.nparts + pi) * (rows * cw);
}

// A wave's rows (lane: row 32 wave + lr of the tile, columns 32 t + 8 (e / 4) + 4
// lh + e % 4 of the pass) divided and stored, or their totals as a part.
template <int CT, int NW>
__device__ __forceinline__ void store_rows(const DirectArgs& a, int bh, int pass, int tile, int pi, int wave,
                                           const double (&zt)[CT][16], double dsum) {
  constexpr int kRows = 32 * NW;
  const int lane = threadIdx.x & 63, lr = lane & 31, lh = lane >> 5;
  const int i = tile * kRows + 32 * wave + lr, c0 = pass * CT * 32 + 4 * lh;
  if (a.nparts == 1) {
    const double inv = 1.0 / dsum;
    if (i >= a.n) return;
    float* __restrict__ zr = a.z + (static_cast<size_t>(bh) * a.n + i) * a.d;
#pragma unroll
    for (int t = 0; t < CT; ++t)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const double* __restrict__ q = &zt[t][4 * g];
        store4(zr, c0 + 32 * t + 8 * g, a.d, static_cast<float>(q[0] * inv), static_cast<float>(q[1] * inv),
               static_cast<float>(q[2] * inv), static_cast<float>(q[3] * inv));
      }
    if (pass == 0 && lh == 0 && a.den) a.den[static_cast<size_t>(bh) * a.n + i] = dsum;
  } else {
    double* __restrict__ part = part_of<CT, NW>(a, bh, pass, tile, pi) + 32 * wave + lr;
#pragma unroll
    for (int t = 0; t < CT; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) part[(32 * t + 8 * (e >> 2) + 4 * lh + (e & 3)) * kRows] = zt[t][e];
    if (lh == 0) part[CT * 32 * kRows] = dsum;
  }
}

// The 32 rows of wave w of k_direct's work-group over the key blocks [b0, b1),
// stored; the rows' denominators in den [32].  Every wave of the work-group calls
// it: phi(q) of the rows goes to LDS (xs, 2 KiB a k step), the waves take the key
// blocks in turn, each forming the keys' features, whose registers are the A
// operands of S, and wave 0 adds the waves' totals.  Few registers are held at a
// time: the kernel's allocation is the main loop's.  Bound by the fp32 matrix cores
// (the keys' projections are formed once per 32 rows): 96 heads, n = 2048, m = 128,
// d = 64, every row 8.1 ms, 0.58 by the fp16 products.
template <typename TV, int KS, int CT, int NW>
__device__ __forceinline__ void exact_rows(const DirectArgs& a, float4* __restrict__ xs, double* __restrict__ den,
                                           int bh, int pass, int tile, int pi, int w, int b0, int b1) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 31, lh = lane >> 5, n = a.n, d = a.d, h = bh % a.H;
  // (trigonometric map: the tiles of sines, then of cosines)
  const bool trf = a.kind == kFeatTrf;
  const int ksp = trf ? KS / 2 : KS, ftiles = (ksp + 1) / 2, all = trf ? 2 * ftiles : ftiles;
  const size_t hb = static_cast<size_t>(bh) * a.nblk, hn = static_cast<size_t>(bh) * n;
  const float* __restrict__ Wh = a.W + static_cast<size_t>(h) * a.m * d;
  const TV* __restrict__ q = static_cast<const TV*>(a.q) + hn * d;
  const TV* __restrict__ k = static_cast<const TV*>(a.k) + hn * d;
  const TV* __restrict__ v = static_cast<const TV*>(a.v) + hn * d;
  const float* __restrict__ ct = a.ctab + static_cast<size_t>(h) * ctab_stride(n);
  const int ct0 = kCPad + n - 1;
  const int wrow0 = (tile * NW + w) * 32, i = wrow0 + lr;
  int wlo, whi;
  {
    const int2 br = head_range(a.crange + static_cast<size_t>(h) * ctab_chunks(n), ctab_chunks(n), lane);
    key_blocks(br, n, wrow0, min(wrow0 + 32, n) - 1, wlo, whi);
  }
  const int lo = max(b0, wlo), hi = min(b1, whi);
  float f[16];
  const int qp = a.qpow[(hb + (wrow0 >> 5)) * kBlk + lr];
  __syncthreads();  // xs and den are free
  for (int ti = wave; ti < all; ti += NW) {
    const bool cosines = ti >= ftiles;
    const int tt = cosines ? ti - ftiles : ti;
    exact_features(a, q + static_cast<size_t>(min(i, n - 1)) * d, i < n, Wh, tt, cosines, qp, f);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if (2 * tt + j >= ksp) continue;  // uniform
      float4* __restrict__ o = xs + ((2 * tt + j + (cosines ? ksp : 0)) * kFragLanes + lane) * 2;
      o[0] = make_float4(f[8 * j], f[8 * j + 1], f[8 * j + 2], f[8 * j + 3]);
      o[1] = make_float4(f[8 * j + 4], f[8 * j + 5], f[8 * j + 6], f[8 * j + 7]);
    }
  }
  __syncthreads();
  double zt[CT][16], dsum = 0.0;
#pragma unroll
  for (int t = 0; t < CT; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) zt[t][e] = 0.0;
#pragma unroll 1
  for (int blk = lo + wave; blk < hi; blk += NW) {
    const float* __restrict__ rec = a.krec + (hb + blk) * kRecWords;
    // (S is at most 2^68: keys down to 2^-140 of the block's largest stand beside it)
    const int pw = __float_as_int(rec[kRecE]) - 2 * kRecBias, vexp = __float_as_int(rec[kRecV]);
    const int key = 32 * blk + lr;
    floatx16 s = zero16();
#pragma unroll 1
    for (int ti = 0; ti < all; ++ti) {
      const bool cosines = ti >= ftiles;
      const int tt = cosines ? ti - ftiles : ti;
      exact_features(a, k + static_cast<size_t>(min(key, n - 1)) * d, key < n, Wh, tt, cosines, pw, f);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if (2 * tt + j >= ksp) continue;  // uniform
        const float4* __restrict__ o = xs + ((2 * tt + j + (cosines ? ksp : 0)) * kFragLanes + lane) * 2;
        const float4 u = o[0], y = o[1];
        const float x8[8] = {u.x, u.y, u.z, u.w, y.x, y.y, y.z, y.w};
#pragma unroll
        for (int t = 0; t < 8; ++t) s = mfma_f32(f[8 * j + t], x8[t], s);
      }
    }
    // lane: row i, keys 8 (e / 4) + 4 lh + e % 4 (groups of four: few loads in
    // flight, few registers); P over the power of its row's largest, as S c may
    // leave fp32's range
    const int j0 = 32 * blk + 4 * lh;
    auto c_of = [&](int e) {
      const int j = j0 + 8 * (e >> 2) + (e & 3);
      return j < n ? at_bytes(ct, static_cast<uint32_t>(j - i + ct0) * 4u) : 0.f;
    };
    int ex = -1000;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float c = c_of(e);
      if (s[e] != 0.f && c > 0.f)
        ex = max(ex, __builtin_amdgcn_frexp_expf(s[e]) + __builtin_amdgcn_frexp_expf(c));
      if (e % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    ex = max(ex, __shfl_xor(ex, 32));
    if (ex == -1000) ex = 0;
    asm volatile("" ::: "memory");  // (c is read again, not held)
    float ds = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float c = c_of(e), mant = __builtin_amdgcn_frexp_mantf(s[e]) * __builtin_amdgcn_frexp_mantf(c);
      s[e] = ldexpf(mant, __builtin_amdgcn_frexp_expf(s[e]) + __builtin_amdgcn_frexp_expf(c) - ex);
      ds += s[e];
      if (e % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    dsum = fma(static_cast<double>(ds), exp2_int(pw + ex), dsum);
    const double zs = exp2_int(pw + vexp + ex);
#pragma unroll
    for (int t = 0; t < CT; ++t) {
      const int col = (pass * CT + t) * 32 + lr;
      floatx16 zc = zero16();
#pragma unroll
      for (int g = 0; g < 4; ++g) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int j = j0 + 8 * g + r;
          const uint32_t at = static_cast<uint32_t>(min(j, n - 1) * d + min(col, d - 1)) * sizeof(TV);
          float vv = j < n && col < d ? to_f32(at_bytes(v, at)) : 0.f;
          vv = isfinite(vv) ? ldexpf(vv, -vexp) : 0.f;  // (the others: k_direct)
          zc = mfma_f32(vv, s[4 * g + r], zc);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) zt[t][e] = fma(static_cast<double>(zc[e]), zs, zt[t][e]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  dsum += __shfl_xor(dsum, 32);
  double* __restrict__ red = reinterpret_cast<double*>(xs) + lane;
  static_assert(CT * 16 * 64 * sizeof(double) <= 16384, "totals: the 16 KiB that every instance holds");
#pragma unroll 1
  for (int src = 1; src < NW; ++src) {
    __syncthreads();  // xs / the previous wave's totals are consumed
    if (wave == src) {
#pragma unroll
      for (int t = 0; t < CT; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) red[(t * 16 + e) * 64] = zt[t][e];
      if (lh == 0) den[lr] = dsum;
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int t = 0; t < CT; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) zt[t][e] += red[(t * 16 + e) * 64];
      dsum += den[lr];
    }
  }
  __syncthreads();
  if (wave == 0) {
    if (lh == 0) den[lr] = dsum;
    store_rows<CT, NW>(a, bh, pass, tile, pi, w, zt, dsum);
  }
  __syncthreads();
}

}  // namespace krpe
