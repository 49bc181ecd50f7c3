// The backward pass of the heads whose rows the forward pass evaluated in fp32
// (direct_args.hpp): the same gradients (bwd_direct.hip) with phi formed again from
// q, k and W and every product on the fp32 matrix cores.  With fq, fk the features
// over their positions' powers, D_i in units of the query's, and
//
//   w_ij = c_{j-i} 2^(power of k_j) / D_i,   T_ij = (dz_i.v_j - dz_i.z_i) w_ij,
//
// dv_j = sum_i (fq_i.fk_j w_ij) dz_i, the sums of the diagonals of (fq_i.fk_j) T_ij, and
// (dphi o phi)(q_i) = fq_i o sum_j T_ij fk_j, (dphi o phi)(k_j) = fk_j o sum_i T_ij fq_i:
// no factor of these leaves fp32's range where the gradients do not.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "bwd_exact.hpp"
#include "common.hpp"
#include "direct_exact.hpp"
#include "features.hpp"
#include "wprod.hpp"

namespace krpe {

// Rare; launched with every backward pass and left at once where no head is
// flagged (4.8 us).  Work-group: 128 rows of one head's queries
// (dq) or keys (dk, dv, diagonals), each wave its own 32, over the key blocks of
// their range, whose features the waves form together.
template <typename TX, int KS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1))) void k_bwd_exact(BwdExactArgs a) {
  constexpr int NW = 4, kTiles = KS / 2, kDT = kMaxD / 32, kDS = 33;
  __shared__ float4 ys[KS * kFragLanes * 2];
  __shared__ float diag[NW][64 * kDS];
  const DirectArgs& f = a.f;
  if (f.flag[f.BH] == 0u) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 31, lh = lane >> 5, n = f.n, d = f.d;
  const int tiles = (n + 32 * NW - 1) / (32 * NW), chunks = ctab_chunks(n), dts = (d + 31) / 32;
  const bool vd = d % 8 == 0;
  for (int e = lane; e < 64 * kDS; e += 64) diag[wave][e] = 0.f;
  for (int item = blockIdx.x; item < f.BH * 2 * tiles; item += gridDim.x) {
    const int tile = item % tiles, bh = item / tiles / 2, h = bh % f.H;
    const bool keys = (item / tiles) % 2 != 0;  // rows: keys
    if (f.flag[bh] == 0u) continue;  // uniform
    const size_t hn = static_cast<size_t>(bh) * n, hb = static_cast<size_t>(bh) * f.nblk;
    const TX* __restrict__ q = static_cast<const TX*>(f.q) + hn * d;
    const TX* __restrict__ k = static_cast<const TX*>(f.k) + hn * d;
    const TX* __restrict__ v = static_cast<const TX*>(f.v) + hn * d;
    const float* __restrict__ dz = a.dz + hn * d;
    const float* __restrict__ z = a.z + hn * d;
    const float* __restrict__ Wh = f.W + static_cast<size_t>(h) * f.m * d;
    const float* __restrict__ ct = (keys ? a.crev : f.ctab) + static_cast<size_t>(h) * ctab_stride(n);
    const int2 br = head_range((keys ? a.rrange : f.crange) + static_cast<size_t>(h) * chunks, chunks, lane);
    const int row0 = tile * 32 * NW, wrow0 = row0 + 32 * wave, r = wrow0 + lr, rc = min(r, n - 1);
    int b0, b1, wlo = 0, whi = 0;
    key_blocks(br, n, row0, min(row0 + 32 * NW, n) - 1, b0, b1);
    if (wrow0 < n) key_blocks(br, n, wrow0, min(wrow0 + 32, n) - 1, wlo, whi);
    // 1 / D_i = mant 2^ex and -dz_i.z_i of a query
    auto query = [&](int i, float& mant, int& ex, float& gamma) {
      const double inv = 1.0 / a.den[hn + i];
      const bool ok = isfinite(inv) && inv != 0.0;
      ex = ok ? ilogb(inv) : 0;
      mant = static_cast<float>(ok ? inv * exp2_int(-ex) : inv);
      double dot = 0.0;
      for (int c = lh; c < d; c += 2)
        dot = fma(static_cast<double>(dz[static_cast<size_t>(i) * d + c]), static_cast<double>(z[static_cast<size_t>(i) * d + c]), dot);
      gamma = static_cast<float>(-(dot + __shfl_xor(dot, 32)));
    };
    float x[KS][8], ft[16];
    auto put = [&](int t) {  // ft to ys as k steps 2 t and 2 t + 1
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        float4* __restrict__ o = ys + ((2 * t + j) * kFragLanes + lane) * 2;
        o[0] = make_float4(ft[8 * j], ft[8 * j + 1], ft[8 * j + 2], ft[8 * j + 3]);
        o[1] = make_float4(ft[8 * j + 4], ft[8 * j + 5], ft[8 * j + 6], ft[8 * j + 7]);
      }
    };
    float rmant = 0.f, rgamma = 0.f;
    int rex = 0;  // of 1 / D_r, or the power of phi(k_r)
    // (the waves in turn, through ys: its own features formed in an unrolled
    // loop take a wave's registers many times over)
    for (int u = 0; u < NW; ++u) {
      __syncthreads();  // ys is free
      if (u != wave || wrow0 >= n) continue;
      const int pw = (keys ? a.kpow : f.qpow)[hb * kBlk + r];
#pragma unroll 1
      for (int t = 0; t < kTiles; ++t) {
        exact_features(f, (keys ? k : q) + static_cast<size_t>(rc) * d, r < n, Wh, t, false, pw, ft);
        put(t);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const float4 y = ys[(ks * kFragLanes + lane) * 2], y1 = ys[(ks * kFragLanes + lane) * 2 + 1];
        x[ks][0] = y.x, x[ks][1] = y.y, x[ks][2] = y.z, x[ks][3] = y.w;
        x[ks][4] = y1.x, x[ks][5] = y1.y, x[ks][6] = y1.z, x[ks][7] = y1.w;
      }
      if (keys)
        rex = pw;
      else
        query(rc, rmant, rex, rgamma);
    }
    floatx16 g[kTiles], dvt[kDT];
#pragma unroll
    for (int t = 0; t < kTiles; ++t) g[t] = zero16();
#pragma unroll
    for (int t = 0; t < kDT; ++t) dvt[t] = zero16();
    float carry = 0.f;
    for (int blk = b0; blk < b1; ++blk) {
      const int key = 32 * blk + lr, kc = min(key, n - 1);
      __syncthreads();  // the previous block's features are consumed
      {
        const int pw = (keys ? f.qpow : a.kpow)[hb * kBlk + key];
        for (int t = wave; t < kTiles; t += NW) {
          exact_features(f, (keys ? q : k) + static_cast<size_t>(kc) * d, key < n, Wh, t, false, pw, ft);
          put(t);
        }
      }
      __syncthreads();
      if (blk < wlo || blk >= whi) continue;  // uniform per wave
      float kmant = 0.f, kgamma = 0.f;
      int kex = 0;
      if (keys)
        query(kc, kmant, kex, kgamma);
      else
        kex = a.kpow[hb * kBlk + key];
      // dz.v: lane row r, keys 8 (e / 4) + 4 lh + e % 4
      floatx16 rr = zero16();
      for (int c = 0; c < d; c += 16) {
        const int c8 = c + 8 * lh;
        float av[8], bv[8];
        if (keys) {
          load8(dz + static_cast<size_t>(kc) * d + c8, d - c8, vd, av);
          load8(v + static_cast<size_t>(rc) * d + c8, d - c8, vd, bv);
        } else {
          load8(v + static_cast<size_t>(kc) * d + c8, d - c8, vd, av);
          load8(dz + static_cast<size_t>(rc) * d + c8, d - c8, vd, bv);
        }
#pragma unroll
        for (int t = 0; t < 8; ++t) rr = mfma_f32(av[t], bv[t], rr);
      }
      float w[16], w0[16];  // with and without c
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int ke = 8 * (e >> 2) + 4 * lh + (e & 3), j = 32 * blk + ke;
        const float km = __shfl(kmant, ke), kg = __shfl(kgamma, ke);
        const int kx = __shfl(kex, ke);
        const bool in = j < n && r < n;
        const float ce = at_bytes(ct, static_cast<uint32_t>(j - r + kCPad + n - 1) * 4u), c = in ? ce : 0.f;
        // (a masked key reaches no row)
        rr[e] = c == 0.f ? 0.f : rr[e] + (keys ? kg : rgamma);
        const float mant = keys ? km : rmant;
        w0[e] = in ? ldexpf(mant, kx + rex) : 0.f;
        w[e] = c == 0.f ? 0.f : ldexpf(mant * c, kx + rex);
      }
      if (keys) {
        floatx16 s = zero16();
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const float4 u = ys[(ks * kFragLanes + lane) * 2], y = ys[(ks * kFragLanes + lane) * 2 + 1];
          const float y8[8] = {u.x, u.y, u.z, u.w, y.x, y.y, y.z, y.w};
#pragma unroll
          for (int t = 0; t < 8; ++t) s = mfma_f32(y8[t], x[ks][t], s);
          if (ks % 2 == 1) __builtin_amdgcn_sched_barrier(0);
        }
        if (a.pdc) {
          // as k_direct's: entry (key) of diagonal 32 + row - key
          float* __restrict__ win = &diag[wave][(32 + lr - 4 * lh) * kDS + 4 * lh];
#pragma unroll
          for (int e = 0; e < 16; ++e) win[(8 * (e >> 2) + (e & 3)) * (1 - kDS)] = s[e] * w0[e] * rr[e];
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          const float* __restrict__ dl = &diag[wave][lane * kDS];
          float up = __shfl(carry, lr);
          up = lh == 1 ? up : 0.f;
          #pragma unroll 8
          for (int t = 0; t < 32; ++t) up += dl[t];
          if (lh == 1) a.pdc[((hb + (wrow0 >> 5)) * (f.nblk + 1) + blk) * 32 + lr] = up;
          carry = up;
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          __builtin_amdgcn_wave_barrier();
        }
#pragma unroll
        for (int t = 0; t < kDT; ++t) {
          if (t >= dts) continue;  // uniform
          const int col = 32 * t + lr;
          floatx16 zc = zero16();
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const int j = 32 * blk + 8 * (e >> 2) + 4 * lh + (e & 3);
            const float y = at_bytes(dz, static_cast<uint32_t>(min(j, n - 1) * d + min(col, d - 1)) * 4u);
            zc = mfma_f32(j < n && col < d ? y : 0.f, s[e] * w[e], zc);
            if (e % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // (few loads in flight, few registers; below too)
          }
          dvt[t] += zc;
        }
      }
      // the keys' features as columns: feature 32 t + lr, position key(e, lh)
      const float* __restrict__ yf = reinterpret_cast<const float*>(ys);
      const int half = (lr >> 2) & 1, slot = 4 * ((lr >> 3) & 1) + (lr & 3);
#pragma unroll
      for (int t = 0; t < kTiles; ++t) {
        floatx16 zc = zero16();
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int ke = 8 * (e >> 2) + 4 * lh + (e & 3);
          const float y = yf[((2 * t + (lr >> 4)) * kFragLanes + ke + 32 * half) * 8 + slot];
          zc = mfma_f32(y, rr[e] * w[e], zc);
        }
        g[t] += zc;
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (keys && a.pdc && lh == 0 && whi > wlo)
      a.pdc[((hb + (wrow0 >> 5)) * (f.nblk + 1) + whi) * 32 + lr] = carry;
    // p = dphi o phi, dx = p W - ..: p through ys, the waves in turn again
    float sum = 0.f;
#pragma unroll
    for (int t = 0; t < kTiles; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        g[t][e] *= x[2 * t + (e >> 3)][e & 7];
        sum += g[t][e];
      }
    sum += __shfl_xor(sum, 32);
    floatx16 acc[kDT];
#pragma unroll
    for (int u = 0; u < kDT; ++u) acc[u] = zero16();
    float* __restrict__ pf = reinterpret_cast<float*>(ys) + lane;
    for (int u = 0; u < NW; ++u) {
      __syncthreads();
      if (u != wave || wrow0 >= n) continue;
#pragma unroll
      for (int t = 0; t < kTiles; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) pf[(16 * t + e) * 64] = g[t][e];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll 4
      for (int te = 0; te < 16 * kTiles; ++te) {
        const int l = 8 * (te >> 2) + 4 * lh + (te & 3);  // feature of register te % 16 of tile te / 16
        const float pv = pf[te * 64];
#pragma unroll
        for (int c = 0; c < kDT; ++c) {
          const int col = 32 * c + lr;
          const float y = at_bytes(Wh, static_cast<uint32_t>(min(l, f.m - 1) * d + min(col, d - 1)) * 4u);
          if (c < dts) acc[c] = mfma_f32(l < f.m && col < d ? y : 0.f, pv, acc[c]);
        }
      }
    }
    if (wrow0 >= n) continue;  // uniform per wave; (the other waves meet it at the next item's barriers)
    const size_t at = (hn + rc) * d;
    store_gradient<TX, kDT>((keys ? k : q) + static_cast<size_t>(rc) * d, acc, sum, (keys ? a.dk : a.dq) + at, r < n, d,
                            f.nprf);
    if (keys && r < n) {
#pragma unroll
      for (int t = 0; t < kDT; ++t)
#pragma unroll
        for (int gq = 0; gq < 4; ++gq)
          store4(a.dv + at, 32 * t + 8 * gq + 4 * lh, d, dvt[t][4 * gq], dvt[t][4 * gq + 1], dvt[t][4 * gq + 2],
                 dvt[t][4 * gq + 3]);
    }
  }
}

namespace {
template <typename TX>
hipError_t go(const BwdExactArgs& a, int ks, hipStream_t st) {
  const long long items = 2LL * a.f.BH * ((a.f.n + 127) / 128);
  const dim3 grid(static_cast<unsigned>(items < 512 ? items : 512)), block(256);
  switch (ks) {
    case 4: hipLaunchKernelGGL((k_bwd_exact<TX, 4>), grid, block, 0, st, a); break;
    case 8: hipLaunchKernelGGL((k_bwd_exact<TX, 8>), grid, block, 0, st, a); break;
    case 16: hipLaunchKernelGGL((k_bwd_exact<TX, 16>), grid, block, 0, st, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
}  // namespace

hipError_t launch_bwd_exact(const BwdExactArgs& a, int ks, bool bf16, hipStream_t st) {
  return bf16 ? go<uint16_t>(a, ks, st) : go<float>(a, ks, st);
}

}  // namespace krpe
