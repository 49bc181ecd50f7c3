// The backward pass on the direct route.  With P_ij = phi(q_i).phi(k_j) c_{j-i},
// D_i = sum_j P_ij, Gh_i = dz_i / D_i, gamma_i = -(dz_i.z_i) / D_i and
// R_ij = (Gh_i.v_j + gamma_i) c_{j-i}, the gradients of L = sum(dz z) are
//
//   dv_j = sum_i P_ij Gh_i           dphi(q_i) = sum_j R_ij phi(k_j)
//   dphi(k_j) = sum_i R_ij phi(q_i)  db_t = c_t sum_i (R_ij / c_t) phi(q_i).phi(k_j), j = i + t
//   dx = (dphi o phi) W - x rowsum(dphi o phi)     (through the row norm with NPRF)
//
// the first three weighted products (wprod.hpp) with the columns gamma and 1
// appended to Gh and v; the last a by-product of dv's, which forms
// phi(q_i).phi(k_j) and takes the other factor as a second product.  phi(q_i)
// stands without its power of two throughout: D_i is then in the same units
// and the power cancels.  Launches: the forward's two, k_bwd_ops (operands from
// dz, z, D and v), k_bwd_exact (the heads that the forward pass flagged, which the
// others then skip: bwd_exact.hip), k_direct for dv, k_db, k_turn (phi as Z operands,
// W's terms), k_direct and k_feature_grad for dq and for dk.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <type_traits>

#include "common.hpp"
#include "bwd_exact.hpp"
#include "direct_kernel.hpp"
#include "launch.hpp"
#include "wprod.hpp"

namespace krpe {

// ------------------------------------------------------------- operands --
struct OpsArgs {
  const void* v;
  const float *dz, *z;
  const double* den;
  const int* kpow;
  const float* krec;  // the forward's records (powers of v)
  uint4 *gs, *vs, *gz;
  float *reca, *recb, *recc, *recd;
  int *gpow, *vpow;
  int BH, n, nblk, d, ks2, ct_total, tiles;
};

// 64 positions of one (batch, head), wave w its 32-position block; source 0:
// Gh and gamma (S and Z fragments, records of dv's and dphi(k)'s keys), source
// 1: [v, 1] (S fragments, records of dphi(q)'s keys).  The 1 is stored as 2^sv, the
// power of the head's largest value, and gamma over it, so that neither column
// is far from the others whatever the values' scale.  Gh as dv's Z operand is taken
// times the power of D_i and dv's records over it: P_ij / D_i is a share of row i,
// while P_ij alone differs between the rows of a block by all that D does.
template <typename TV>
__global__ __launch_bounds__(128) void k_bwd_ops(OpsArgs a) {
  constexpr int XS = kMaxD + 16 + 4;
  __shared__ __align__(16) float rows[2][32][XS];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 31, lh = lane >> 5, n = a.n, d = a.d;
  int b = blockIdx.x;
  const int pt = b % a.tiles;
  b /= a.tiles;
  const int bh = b % a.BH, src = b / a.BH, blk = 2 * pt + wave;
  if (blk >= a.nblk) return;  // uniform per wave; waves share nothing here
  const size_t block = static_cast<size_t>(bh) * a.nblk + blk;
  float(*__restrict__ row)[XS] = rows[wave];
  int sv = -400;
  for (int j = lane; j < a.nblk; j += 64)
    sv = max(sv, __float_as_int(a.krec[(static_cast<size_t>(bh) * a.nblk + j) * kRecWords + kRecV]) + 15);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) sv = max(sv, __shfl_xor(sv, off));
  int dp = 0;  // power of D_i
  // rows of dz or v to LDS (zeros past n and past d)
  const size_t at = (static_cast<size_t>(bh) * n + 32 * blk) * d;
  const int live = min(32, n - 32 * blk);
  const bool vec = d % 8 == 0;  // rows 16-byte aligned, whole groups of 8
  for (int e = lane; e < 32 * 2 * a.ks2; e += 64) {
    const int r = e / (2 * a.ks2), c8 = 8 * (e % (2 * a.ks2));
    float v8[8];
    const size_t o = at + static_cast<size_t>(min(r, live - 1)) * d + c8;
    const int count = r < live ? d - c8 : 0;
    if (src == 0)
      load8(a.dz + o, count, vec, v8);
    else
      load8(static_cast<const TV*>(a.v) + o, count, vec, v8);
    *reinterpret_cast<float4*>(&row[r][c8]) = make_float4(v8[0], v8[1], v8[2], v8[3]);
    *reinterpret_cast<float4*>(&row[r][c8 + 4]) = make_float4(v8[4], v8[5], v8[6], v8[7]);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const bool ok = lr < live;
  if (src == 0) {
    // lane half lh takes the groups of 4 columns 2 g + lh of its row
    const size_t i = static_cast<size_t>(bh) * n + 32 * blk + min(lr, live - 1);
    const double den = a.den[i], inv = ok ? 1.0 / den : 0.0;
    if (ok && isfinite(den) && den != 0.0) dp = ilogb(den) + 1;
    const float* __restrict__ zr = a.z + i * d;
    double dot = 0.0;
    for (int c = 4 * lh; c < d; c += 8) {
      float4 g = *reinterpret_cast<const float4*>(&row[lr][c]);
      float zv[4];
      if (d % 4 == 0) {
        const float4 t = *reinterpret_cast<const float4*>(zr + c);
        zv[0] = t.x, zv[1] = t.y, zv[2] = t.z, zv[3] = t.w;
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) zv[j] = c + j < d ? zr[c + j] : 0.f;
      }
      dot = fma(static_cast<double>(g.x), static_cast<double>(zv[0]), dot);
      dot = fma(static_cast<double>(g.y), static_cast<double>(zv[1]), dot);
      dot = fma(static_cast<double>(g.z), static_cast<double>(zv[2]), dot);
      dot = fma(static_cast<double>(g.w), static_cast<double>(zv[3]), dot);
      g.x = static_cast<float>(g.x * inv), g.y = static_cast<float>(g.y * inv);
      g.z = static_cast<float>(g.z * inv), g.w = static_cast<float>(g.w * inv);
      *reinterpret_cast<float4*>(&row[lr][c]) = g;
    }
    dot += __shfl_xor(dot, 32);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();  // (the group of 4 that holds column d is rewritten above when d % 4 != 0)
    if (lh == 0) row[lr][d] = ok ? static_cast<float>(-dot * inv * exp2_int(-sv)) : 0.f;
  } else if (lh == 0) {
    row[lr][d] = ok ? ldexpf(1.f, sv) : 0.f;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  // S fragments with the position's power
  float mx = 0.f;
  for (int ks = 0; ks < a.ks2; ++ks)
#pragma unroll
    for (int t = 0; t < 8; ++t) mx = fmaxf(mx, fabsf(row[lr][16 * ks + 8 * (t >> 2) + 4 * lh + (t & 3)]));
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  const bool any = mx > 0.f;
  const int ex = __builtin_amdgcn_frexp_expf(mx) - 15;
  uint4* __restrict__ so = (src == 0 ? a.gs : a.vs) + block * a.ks2 * 2 * kFragLanes + lane;
  for (int ks = 0; ks < a.ks2; ++ks) {
    float v8[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) v8[t] = ldexpf(row[lr][16 * ks + 8 * (t >> 2) + 4 * lh + (t & 3)], -ex);
    uint4 hh, ll;
    split_f16x8(v8, kLoScale, hh, ll);
    so[(ks * 2 + 0) * kFragLanes] = hh;
    so[(ks * 2 + 1) * kFragLanes] = ll;
  }
  // records: the power of the keys' product with its Z operand's
  const int kp = src == 0 ? ex : ex + a.kpow[block * kBlk + lr];
  int E = any ? kp : -800;
#pragma unroll
  for (int off = 16; off > 0; off >>= 1) E = max(E, __shfl_xor(E, off));
  float* __restrict__ rec = (src == 0 ? a.recc : a.recb) + block * kRecWords;
  if (lh == 0) {
    rec[lr] = any ? ldexpf(1.f, kp - E - kRecBias) : 0.f;
    (src == 0 ? a.gpow : a.vpow)[block * kBlk + lr] = ex;
  }
  if (lane == 0) {
    rec[kRecE] = __int_as_float(E + kRecBias);
    rec[kRecV] = __int_as_float(0);
  }
  if (src == 1) return;
  // Gh over the power of 1 / D_i as Z fragments with the block's power
  float gm = 0.f;
  for (int ct = 0; ct < a.ct_total; ++ct) {
    const int c = 32 * ct + lr;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int r = 8 * (e >> 2) + 4 * lh + (e & 3);
      const float g = ldexpf(row[r][min(c, d)], __shfl(dp, r));
      gm = fmaxf(gm, c < d ? fabsf(g) : 0.f);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) gm = fmaxf(gm, __shfl_xor(gm, off));
  const int gx = __builtin_amdgcn_frexp_expf(gm) - 15;
  uint4* __restrict__ zo = a.gz + block * a.ct_total * 4 * kFragLanes + lane;
  for (int ct = 0; ct < a.ct_total; ++ct) {
    const int c = 32 * ct + lr;
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2) {
      float v8[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int r = 16 * k2 + 8 * (t >> 2) + 4 * lh + (t & 3);
        const float g = ldexpf(row[r][min(c, d)], __shfl(dp, r) - gx);
        v8[t] = c < d ? g : 0.f;
      }
      uint4 hh, ll;
      split_f16x8(v8, kLoScale, hh, ll);
      zo[((ct * 2 + k2) * 2 + 0) * kFragLanes] = hh;
      zo[((ct * 2 + k2) * 2 + 1) * kFragLanes] = ll;
    }
  }
  // dv's keys: phi(q) without its power, over D_i's; the diagonal sums' with it
  auto record = [&](float* __restrict__ r, int p, bool has, int v) {
    int e = has ? p : -800;
#pragma unroll
    for (int off = 16; off > 0; off >>= 1) e = max(e, __shfl_xor(e, off));
    if (lh == 0) r[lr] = has ? ldexpf(1.f, p - e - kRecBias) : 0.f;
    if (lane == 0) {
      r[kRecE] = __int_as_float(e + kRecBias);
      r[kRecV] = __int_as_float(v);
    }
  };
  record(a.reca + block * kRecWords, -dp, ok, gx);
  record(a.recd + block * kRecWords, ex + dp, any, 0);
}

// W as Z fragments in three bf16 terms: [H][ks][d tile][3][64], lane: column
// 32 dt + lr, features 16 ks + 8 (t / 4) + 4 lh + t % 4.  One wave a fragment.
struct WTerms {
  const float* W;
  uint4* wf;
  int H, d, m, KS, dts;
};
__device__ __forceinline__ void wterms(const WTerms& a, int item) {
  const int lane = threadIdx.x & 63, lr = lane & 31, lh = lane >> 5;
  const int dt = item % a.dts, ks = item / a.dts % a.KS, h = item / a.dts / a.KS, c = 32 * dt + lr;
  if (h >= a.H) return;
  float v8[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    const int l = 16 * ks + 8 * (t >> 2) + 4 * lh + (t & 3);
    v8[t] = l < a.m && c < a.d ? a.W[(static_cast<size_t>(h) * a.m + l) * a.d + c] : 0.f;
  }
  uint4 t3[3];
  split_bf16x8(v8, t3);
#pragma unroll
  for (int s = 0; s < 3; ++s) a.wf[(static_cast<size_t>(item) * 3 + s) * kFragLanes + lane] = t3[s];
}

// S fragments of phi turned into Z fragments (the same values; powers are the
// records' matter): one wave per 32 positions x 32 features through LDS.  The
// waves past these form W's terms (a launch of its own took 5 us).
__global__ __launch_bounds__(256) void k_turn(const uint4* __restrict__ s0, const uint4* __restrict__ s1,
                                              uint4* __restrict__ z0, uint4* __restrict__ z1, int KS, int ct_total,
                                              long long waves, long long blocks, WTerms wt) {
  __shared__ uint16_t t[4][2][32][36];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 31, lh = lane >> 5;
  const long long id = static_cast<long long>(blockIdx.x) * 4 + wave;
  if (id >= waves) {  // uniform per wave; waves share nothing
    wterms(wt, static_cast<int>(id - waves));
    return;
  }
  const int ct = static_cast<int>(id % ct_total);
  long long block = id / ct_total;
  const bool second = block >= blocks;
  if (second) block -= blocks;
  const uint4* __restrict__ s = (second ? s1 : s0) + block * KS * 2 * kFragLanes + lane;
  uint4* __restrict__ z = (second ? z1 : z0) + (block * ct_total + ct) * 4 * kFragLanes + lane;
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int ks = 2 * ct + j;
      const uint4 u = ks < KS ? s[(ks * 2 + i) * kFragLanes] : make_uint4(0u, 0u, 0u, 0u);
      const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
      for (int e = 0; e < 8; ++e)
        t[wave][i][16 * j + 8 * (e >> 2) + 4 * lh + (e & 3)][lr] = static_cast<uint16_t>(w[e >> 1] >> (16 * (e & 1)));
    }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint2 a = *reinterpret_cast<const uint2*>(&t[wave][i][lr][16 * k2 + 4 * lh]);
      const uint2 c = *reinterpret_cast<const uint2*>(&t[wave][i][lr][16 * k2 + 8 + 4 * lh]);
      z[(k2 * 2 + i) * kFragLanes] = make_uint4(a.x, a.y, c.x, c.y);
    }
}

// ----------------------------------------------------- feature gradient --
// dx of 32 positions per wave: p = dphi o phi (times the position's power for
// the keys), dx = p W - x sum(p) with six bf16 products per term, and the
// projection of the row norm with NPRF.  dphi is consumed in its fragment
// order, which is the operand order of this product.
template <typename TX, int DT>
__global__ __launch_bounds__(256) void k_feature_grad(const TX* __restrict__ x, const uint4* __restrict__ wf,
                                                      const uint4* __restrict__ phi, const float* __restrict__ dphi,
                                                      const int* __restrict__ pow, const unsigned* __restrict__ flag,
                                                      float* __restrict__ dx, int H, int n, int nblk, int d, int KS,
                                                      int nprf, int BH) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 31, lh = lane >> 5;
  const int tiles = (nblk + 3) / 4;
  const int bh = blockIdx.x / tiles, blk = 4 * (blockIdx.x % tiles) + wave, h = bh % H;
  if (blk >= nblk || flag[bh] != 0u) return;  // uniform per wave; no barrier
  const size_t block = static_cast<size_t>(bh) * nblk + blk;
  const uint4* __restrict__ fp = phi + block * KS * 2 * kFragLanes + lane;
  const float4* __restrict__ gp = reinterpret_cast<const float4*>(dphi) + (block * KS * kFragLanes + lane) * 2;
  const uint4* __restrict__ wp = wf + static_cast<size_t>(h) * KS * DT * 3 * kFragLanes + lane;
  const int pw = pow ? pow[block * kBlk + lr] : 0;
  floatx16 acc[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t) acc[t] = zero16();
  float sum = 0.f;
  for (int ks = 0; ks < KS; ++ks) {
    const uint4 hh = fp[(ks * 2 + 0) * kFragLanes], ll = fp[(ks * 2 + 1) * kFragLanes];
    const float4 g0 = gp[ks * 2 * kFragLanes], g1 = gp[ks * 2 * kFragLanes + 1];
    const uint32_t hw[4] = {hh.x, hh.y, hh.z, hh.w}, lw[4] = {ll.x, ll.y, ll.z, ll.w};
    const float g[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
    float v8[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      v8[t] = g[t] * ldexpf(term_value(hw[t >> 1], lw[t >> 1], t & 1), pw);
      sum += v8[t];
    }
    uint4 p3[3];
    split_bf16x8(v8, p3);
#pragma unroll
    for (int t = 0; t < DT; ++t) {
      uint4 w3[3];
#pragma unroll
      for (int s = 0; s < 3; ++s) w3[s] = wp[((ks * DT + t) * 3 + s) * kFragLanes];
#pragma unroll
      for (int s = 2; s >= 0; --s)
#pragma unroll
        for (int i = 0; i <= s; ++i) acc[t] = mfma_bf16(w3[i], p3[s - i], acc[t]);
    }
  }
  sum += __shfl_xor(sum, 32);
  const int i = 32 * blk + lr;
  const TX* __restrict__ xr = x + (static_cast<size_t>(bh) * n + min(i, n - 1)) * d;
  store_gradient<TX, DT>(xr, acc, sum, dx + (static_cast<size_t>(bh) * n + min(i, n - 1)) * d, i < n, d, nprf);
}

// db_t = c_t x the diagonal sums over the row blocks of every batch entry, in
// fp64.  Entry (jb, slot s, k) of pdc is the sum over t = 32 (jb - s) + k of
// one row block jb (rows j, keys i, t = j - i).  Work-group: 64 offsets t, four
// groups of waves over the (batch, row block) pairs.
__global__ __launch_bounds__(256) void k_db(const float* __restrict__ pdc, const float* __restrict__ ctab,
                                            const int2* __restrict__ rrange, float* __restrict__ db, int B, int H,
                                            int n, int nblk) {
  __shared__ double red[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int h = blockIdx.y, chunks = ctab_chunks(n);
  const int sidx = blockIdx.x * 64 + lane, t = sidx - (n - 1);
  const int2 br = head_range(rrange + static_cast<size_t>(h) * chunks, chunks, lane);
  const int q = t >= 0 ? t / 32 : -((31 - t) / 32), k = t - 32 * q;  // t = 32 q + k, 0 <= k < 32
  double s = 0.0;
  for (int e = wave; e < B * nblk; e += 4) {
    const int bt = e / nblk, jb = e - bt * nblk;
    int lo, hi;
    key_blocks(br, n, 32 * jb, min(32 * jb + 32, n) - 1, lo, hi);
    const int slot = jb - q;
    if (lo < hi && slot >= lo && slot <= hi)
      s += pdc[((static_cast<size_t>(bt) * H + h) * nblk + jb) * (nblk + 1) * 32 + slot * 32 + k];
  }
  red[wave][lane] = s;
  __syncthreads();
  if (wave == 0 && sidx < 2 * n - 1) {
    const float c = ctab[static_cast<size_t>(h) * ctab_stride(n) + kCPad + sidx];
    const double sum = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
    db[static_cast<size_t>(h) * (2 * n - 1) + sidx] = c == 0.f ? 0.f : static_cast<float>(sum * c);
  }
}

// ------------------------------------------------------------ launchers --
namespace {

// Waves per work-group: four, two work-groups per CU; eight, one per CU, where
// the diagonals' LDS leaves room for one only (with more than 128 features
// one wave per SIMD runs anyway).
constexpr int bwd_waves(int MODE, int KS) { return MODE == 2 && KS <= 8 ? 8 : 4; }

template <int MODE, int KS, int KS2, int CT>
hipError_t go(DirectArgs a, hipStream_t st) {
  constexpr int NW = bwd_waves(MODE, KS);
  a.tiles = (a.n + 32 * NW - 1) / (32 * NW);
  const long long blocks = static_cast<long long>(a.BH) * a.passes * a.tiles;
  hipLaunchKernelGGL((k_direct<MODE, 2, KS, KS2, CT, NW>), dim3(static_cast<unsigned>(blocks)), dim3(64 * NW), 0, st, a);
  return hipGetLastError();
}

// dv: rows phi(k), keys phi(q), columns Gh
template <int KS>
hipError_t go_dv(const DirectArgs& a, int ks2, bool db, hipStream_t st) {
  if (a.ct_total == 1) return db ? go<2, KS, 3, 1>(a, st) : go<1, KS, 0, 1>(a, st);
  if (!db) return go<1, KS, 0, 2>(a, st);
  return ks2 <= 3 ? go<2, KS, 3, 2>(a, st) : ks2 <= 5 ? go<2, KS, 5, 2>(a, st) : go<2, KS, 9, 2>(a, st);
}
// dphi: rows and keys of d + 1 contracted columns, columns phi
template <int KS2>
hipError_t go_dphi(const DirectArgs& a, int ct, hipStream_t st) {
  return ct == 2 ? go<1, KS2, 0, 2>(a, st) : go<1, KS2, 0, 4>(a, st);
}

template <typename TX>
hipError_t feature_grad(const void* x, const uint4* wf, const uint4* phi, const float* dphi, const int* pow,
                        const unsigned* flag, float* dx, int BH, int H, int n, int nblk, int d, int KS, bool nprf, hipStream_t st) {
  const dim3 grid(static_cast<unsigned>(static_cast<long long>(BH) * ((nblk + 3) / 4))), block(256);
  const TX* xt = static_cast<const TX*>(x);
  const int np = nprf ? 1 : 0;
  if (d <= 32)
    hipLaunchKernelGGL((k_feature_grad<TX, 1>), grid, block, 0, st, xt, wf, phi, dphi, pow, flag, dx, H, n, nblk, d, KS, np, BH);
  else if (d <= 64)
    hipLaunchKernelGGL((k_feature_grad<TX, 2>), grid, block, 0, st, xt, wf, phi, dphi, pow, flag, dx, H, n, nblk, d, KS, np, BH);
  else
    hipLaunchKernelGGL((k_feature_grad<TX, 4>), grid, block, 0, st, xt, wf, phi, dphi, pow, flag, dx, H, n, nblk, d, KS, np, BH);
  return hipGetLastError();
}

int d_tiles(int d) { return d <= 32 ? 1 : d <= 64 ? 2 : 4; }

}  // namespace

// k steps of phi in the backward products (4, 8 or 16; 0: more than 256 features)
int direct_bwd_ksteps(int m) { return m <= 64 ? 4 : m <= 128 ? 8 : m <= 256 ? 16 : 0; }

DirectBwdLayout direct_bwd_layout(int B, int H, int n, int d, int m) {
  DirectBwdLayout L{};
  const int ks = direct_bwd_ksteps(m);
  L.f = direct_layout(B, H, n, d, ks);
  const size_t bh = static_cast<size_t>(B) * H, nb = static_cast<size_t>(L.f.nblk);
  const int want = (d + 1 + 15) / 16;
  L.ks2 = want <= 3 ? 3 : want <= 5 ? 5 : 9;
  const int ct = ks / 2;  // 2, 4 or 8
  L.ctq = ct == 2 ? 2 : 4;
  L.passq = (ct + L.ctq - 1) / L.ctq;
  size_t off = L.f.total;
  auto take = [&off](size_t bytes) {
    const size_t at = off;
    off = (off + bytes + 255) & ~static_cast<size_t>(255);
    return at;
  };
  constexpr size_t kFrag = kFragLanes * sizeof(uint4);
  L.z = take(bh * n * d * sizeof(float));
  L.den = take(bh * n * sizeof(double));
  L.kpow = take(bh * nb * kBlk * sizeof(int));
  L.crev = take(static_cast<size_t>(H) * ctab_stride(n) * sizeof(float));
  L.rrange = take(static_cast<size_t>(H) * ctab_chunks(n) * sizeof(int2));
  L.gs = take(bh * nb * L.ks2 * 2 * kFrag);
  L.vs = take(bh * nb * L.ks2 * 2 * kFrag);
  L.gz = take(bh * nb * L.f.ct_total * 4 * kFrag);
  L.reca = take(bh * nb * kRecWords * sizeof(float));
  L.recb = take(bh * nb * kRecWords * sizeof(float));
  L.recc = take(bh * nb * kRecWords * sizeof(float));
  L.recd = take(bh * nb * kRecWords * sizeof(float));
  L.gpow = take(bh * nb * kBlk * sizeof(int));
  L.vpow = take(bh * nb * kBlk * sizeof(int));
  L.wf = take(static_cast<size_t>(H) * ks * d_tiles(d) * 3 * kFrag);
  // the diagonal sums are read before phi's Z operands and dphi are written: they
  // take the same place (they grow with n^2, the others with n m)
  const size_t phz = bh * nb * L.passq * L.ctq * 4 * kFrag, dphi = bh * nb * ks * kFragLanes * 8 * sizeof(float);
  const size_t pdc = bh * nb * (nb + 1) * 32 * sizeof(float);
  L.zq = L.pdc = off;
  L.zk = L.zq + phz;
  L.dphi = L.zk + phz;
  take(pdc > 2 * phz + dphi ? pdc : 2 * phz + dphi);
  L.total = off;
  return L;
}

hipError_t launch_direct_bwd(const DirectBwdLayout& L, char* w, const void* q, const void* k, const void* v, bool bf16,
                             const float* b, const float* W, const float* dz, float* dq, float* dk, float* dv,
                             float* db, int BH, int H, int n, int d, int m, bool nprf, hipStream_t st) {
  const DirectLayout& F = L.f;
  auto U = [&](size_t o) { return reinterpret_cast<uint4*>(w + o); };
  auto Fl = [&](size_t o) { return reinterpret_cast<float*>(w + o); };
  auto I = [&](size_t o) { return reinterpret_cast<int*>(w + o); };
  int2* rrange = reinterpret_cast<int2*>(w + L.rrange);
  double* den = reinterpret_cast<double*>(w + L.den);
  unsigned* flag = reinterpret_cast<unsigned*>(w + F.flag);
  const int nblk = F.nblk;
  if (hipError_t e = launch_direct_prep(F, w, q, k, v, bf16, b, W, BH, H, n, d, m, nprf, kFeatPrf, I(L.kpow),
                                        Fl(L.crev), rrange, st);
      e != hipSuccess)
    return e;
  if (hipError_t e = launch_direct(F, w, q, k, v, bf16, W, Fl(L.z), den, BH, H, n, d, m, nprf, kFeatPrf, st);
      e != hipSuccess)
    return e;

  OpsArgs o{};
  o.v = v, o.dz = dz, o.z = Fl(L.z), o.den = den, o.kpow = I(L.kpow), o.krec = Fl(F.krec);
  o.gs = U(L.gs), o.vs = U(L.vs), o.gz = U(L.gz);
  o.reca = Fl(L.reca), o.recb = Fl(L.recb), o.recc = Fl(L.recc), o.recd = Fl(L.recd), o.gpow = I(L.gpow), o.vpow = I(L.vpow);
  o.BH = BH, o.n = n, o.nblk = nblk, o.d = d, o.ks2 = L.ks2, o.ct_total = F.ct_total, o.tiles = (nblk + 1) / 2;
  const dim3 ogrid(static_cast<unsigned>(static_cast<long long>(2) * BH * o.tiles));
  if (bf16)
    hipLaunchKernelGGL(k_bwd_ops<uint16_t>, ogrid, dim3(128), 0, st, o);
  else
    hipLaunchKernelGGL(k_bwd_ops<float>, ogrid, dim3(128), 0, st, o);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;

  // the heads whose phi two fp16 terms do not hold (the launches below skip them)
  BwdExactArgs x{};
  direct_exact_args(F, w, q, k, v, bf16, W, BH, H, n, d, m, nprf, kFeatPrf, x.f);
  x.dz = dz, x.z = Fl(L.z), x.den = den, x.kpow = I(L.kpow), x.crev = Fl(L.crev), x.rrange = rrange;
  x.dq = dq, x.dk = dk, x.dv = dv, x.pdc = db ? Fl(L.pdc) : nullptr;
  if (hipError_t e = launch_bwd_exact(x, F.ks, bf16, st); e != hipSuccess) return e;

  DirectArgs a{};
  a.BH = BH, a.H = H, a.n = n, a.nblk = nblk, a.d = d, a.nparts = 1, a.flag = flag;
  a.remap = direct_remap(BH);
  // dv_j = sum_i P_ij Gh_i (rows j, keys i: the reversed table), and the
  // diagonal sums of (v_j.Gh_i + gamma_i) (phi(k_j).phi(q_i))
  a.X = U(F.y), a.Y = U(F.x), a.Z = U(L.gz), a.krec = Fl(L.reca), a.rpow = I(L.kpow);
  a.ctab = Fl(L.crev), a.crange = rrange, a.ct_total = F.ct_total, a.passes = F.passes, a.z = dv, a.ldz = d;
  a.X2 = U(L.vs), a.Y2 = U(L.gs), a.krec2 = Fl(L.recd), a.rpow2 = I(L.vpow), a.pdc = Fl(L.pdc);
  hipError_t e = F.ks == 4   ? go_dv<4>(a, L.ks2, db != nullptr, st)
                 : F.ks == 8 ? go_dv<8>(a, L.ks2, db != nullptr, st)
                             : go_dv<16>(a, L.ks2, db != nullptr, st);
  if (e != hipSuccess) return e;
  if (db) {
    hipLaunchKernelGGL(k_db, dim3(static_cast<unsigned>((2 * n - 1 + 63) / 64), static_cast<unsigned>(H)), dim3(256), 0,
                       st, Fl(L.pdc), Fl(F.ctab), rrange, db, BH / H, H, n, nblk);
    if (e = hipGetLastError(); e != hipSuccess) return e;
  }
  // (not before: its operands take the place of the diagonal sums)
  const int ctt = L.passq * L.ctq, dts = d_tiles(d);
  const long long blocks = static_cast<long long>(BH) * nblk, waves = 2 * blocks * ctt;
  const WTerms wt{W, U(L.wf), H, d, m, F.ks, dts};
  const long long all = waves + static_cast<long long>(H) * F.ks * dts;
  hipLaunchKernelGGL(k_turn, dim3(static_cast<unsigned>((all + 3) / 4)), dim3(256), 0, st, U(F.x), U(F.y), U(L.zq),
                     U(L.zk), F.ks, ctt, waves, blocks, wt);
  if (e = hipGetLastError(); e != hipSuccess) return e;
  auto dphi = [&](const DirectArgs& x) {
    return L.ks2 == 3 ? go_dphi<3>(x, L.ctq, st) : L.ks2 == 5 ? go_dphi<5>(x, L.ctq, st) : go_dphi<9>(x, L.ctq, st);
  };
  auto grad = [&](const void* x, size_t phi, const int* pow, float* dx) {
    return bf16 ? feature_grad<uint16_t>(x, U(L.wf), U(phi), Fl(L.dphi), pow, flag, dx, BH, H, n, nblk, d, F.ks, nprf, st)
                : feature_grad<float>(x, U(L.wf), U(phi), Fl(L.dphi), pow, flag, dx, BH, H, n, nblk, d, F.ks, nprf, st);
  };
  // dphi(q_i) = sum_j R_ij phi(k_j) (rows i, keys j), then dq
  a.X = U(L.gs), a.Y = U(L.vs), a.Z = U(L.zk), a.krec = Fl(L.recb), a.rpow = I(L.gpow);
  a.ctab = Fl(F.ctab), a.crange = reinterpret_cast<const int2*>(w + F.crange);
  a.ct_total = ctt, a.passes = L.passq, a.z = Fl(L.dphi), a.ldz = 0, a.out_ks = F.ks;
  if (e = dphi(a); e != hipSuccess) return e;
  if (e = grad(q, F.x, nullptr, dq); e != hipSuccess) return e;
  // dphi(k_j) = sum_i R_ij phi(q_i) (rows j, keys i), then dk
  a.X = U(L.vs), a.Y = U(L.gs), a.Z = U(L.zq), a.krec = Fl(L.recc), a.rpow = I(L.vpow);
  a.ctab = Fl(L.crev), a.crange = rrange;
  if (e = dphi(a); e != hipSuccess) return e;
  return grad(k, F.y, I(L.kpow), dk);
}

}  // namespace krpe
