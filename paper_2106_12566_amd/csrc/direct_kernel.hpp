// The kernel of the weighted products (wprod.hpp), shared by the direct route
// of the forward pass (direct.hip) and the backward pass (bwd_direct.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "common.hpp"
#include "direct_args.hpp"
#include "direct_exact.hpp"
#include "features.hpp"
#include "wprod.hpp"

namespace krpe {

// --------------------------------------------------------------- direct --
// One work-group: 32 NW consecutive rows of one (batch, head), each wave its
// own 32, over the 32-key blocks of its part of the rows' finite-b range.  A
// block's fragments of phi(k) and v, its strip of c and its record are staged
// to LDS one block ahead by direct loads and shared by the waves; phi(q) stays
// in registers.  Per block and wave: S^T = phi(k) phi(q)^T (lane: row lr, keys
// along the registers), P = S^T 2^(e_j - E) c_{j-i}, P split with the power of
// its row's largest entry, and Z^T = [v]^T P^T (lane: row lr again, so that
// the row's power applies lane by lane), whose fp32 sums over the 32 keys are
// added into fp64 totals; the denominator is the fp32 sum of P added likewise.
// The power of phi(q_i) cancels in z.  The forward pass stores P's small term
// unscaled (its largest entry is at 2^14, terms below 2^-40 of that are lost: the
// row test counts it); the backward's products, whose weights R_ij = (..) / D_i
// differ within a block by all that D does, scale it (2^-51), 16 multiplications
// a block.  A wave skips
// the blocks outside its own rows' range (it still stages and meets the
// barriers).  The forward pass sums the weights of S too (kRowTau's test, 1.5 to 2 %
// of a long call: 1.98 -> 2.01 ms at 96 heads, n = 4096, m = 128); a branch on
// each block's least S instead costs 2.5 to 4 %, and so does holding anything for
// the rows that fail through the loop.

// Whether the work-groups take XCD order: one XCD's L2 then serves the
// work-groups of a head; with few heads the plain order spreads the row tiles,
// whose lengths differ, over the XCDs.
inline bool direct_remap(int BH) { return BH >= 16 || BH % 8 == 0; }

// Has the loads of x complete here: a first use inside the loop would wait
// there, every time, for all outstanding loads, the staged ones too.
template <int N>
__device__ __forceinline__ void keep(uint4 (&x)[N][2]) {
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int s = 0; s < 2; ++s) asm volatile("" : "+v"(x[i][s].x), "+v"(x[i][s].y), "+v"(x[i][s].z), "+v"(x[i][s].w));
}

// s + s1 / kLoScale = Y X^T over KS k steps: Y's fragments are read from LDS
// two steps ahead of their products, up to 8 steps (beyond, X leaves no
// registers for it: at 16 steps it spills, 3.9 -> 5.6 ms at n = 16384).
constexpr int kAheadSteps = 8;
template <int KS>
__device__ __forceinline__ void s_product(const uint4* __restrict__ y, const uint4 (&x)[KS][2], floatx16& s, floatx16& s1) {
  s = zero16();
  s1 = zero16();
  if constexpr (KS > kAheadSteps) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const uint4 yh = y[(ks * 2 + 0) * kFragLanes], yl = y[(ks * 2 + 1) * kFragLanes];
      s = mfma_f16(yh, x[ks][0], s);
      s1 = mfma_f16(yh, x[ks][1], s1);
      s1 = mfma_f16(yl, x[ks][0], s1);
    }
    return;
  }
  uint4 yb[3][2];
#pragma unroll
  for (int ks = 0; ks < 2 && ks < KS; ++ks)
#pragma unroll
    for (int i = 0; i < 2; ++i) yb[ks][i] = y[(ks * 2 + i) * kFragLanes];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    if (ks + 2 < KS) {
#pragma unroll
      for (int i = 0; i < 2; ++i) yb[(ks + 2) % 3][i] = y[((ks + 2) * 2 + i) * kFragLanes];
    }
    s = mfma_f16(yb[ks % 3][0], x[ks][0], s);
    s1 = mfma_f16(yb[ks % 3][0], x[ks][1], s1);
    s1 = mfma_f16(yb[ks % 3][1], x[ks][0], s1);
  }
}
// The order of s_product's reads and products (one scheduling region): kDs LDS
// reads, the products of a step, and so on, with room for the reads of later
// phases.
constexpr int kSchedMfma = 0x8, kSchedDsRead = 0x100;
template <int KS>
__device__ __forceinline__ void s_schedule() {
  __builtin_amdgcn_sched_group_barrier(kSchedDsRead, 4, 0);
  constexpr_for<KS>([&](auto) {
    __builtin_amdgcn_sched_group_barrier(kSchedDsRead, 4, 0);
    __builtin_amdgcn_sched_group_barrier(kSchedMfma, 3, 0);
  });
}

// MODE 0: the forward pass.  MODE 1: the plain product, fp32 totals, rows
// scaled by their powers.  MODE 2: as MODE 1, and the diagonal sums of
// (X2 Y2^T) o (X Y^T) in pass 0 (bwd_direct.hip).
// Waves per SIMD: what the main loop's registers allow (exact_rows would take
// more of them for its loads).
template <int MODE, int KS, int CT>
constexpr int kDirectWaves = MODE == 0 && CT == 1 && KS <= 2 ? 4 : MODE == 0 && KS * CT <= 4 ? 3 : 2;
template <int MODE, int NSZ, int KS, int KS2, int CT, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(kDirectWaves<MODE, KS, CT>))) void k_direct(DirectArgs a) {
  using TV = typename std::conditional<NSZ == 1, uint16_t, float>::type;
  using Total = typename std::conditional<MODE == 0, double, float>::type;
  constexpr int kRows = 32 * NW;
  constexpr int NY = KS * 2, NY2 = MODE == 2 ? KS2 * 2 : 0, NZ = CT * 2 * NSZ;
  constexpr int NF = NY + NY2 + NZ;           // fragments per key block
  constexpr int NC = (kRows + 31 + 63) / 64;  // 64-entry pieces of the c strip (kRows + 31 entries used)
  constexpr int NR = MODE == 2 ? 2 : 1;       // records
  constexpr int kStrip = NC * 64 + NR * kRecWords;
  __shared__ uint4 tiles_lds[2][NF * kFragLanes];
  __shared__ __align__(16) float strip[2][kStrip];
  constexpr float kPLow = MODE > 0 ? kLoScale : 1.f;  // scale of P's small term
  constexpr int kDS = 33;  // floats per diagonal: writes across the lanes and reads fall in distinct banks
  __shared__ float diag[MODE == 2 ? NW : 1][MODE == 2 ? 64 * kDS : 1];
  __shared__ unsigned redo;  // MODE 0: waves whose rows are evaluated again,
  __shared__ double den[MODE == 0 ? 32 : 1];  // and one's denominators
  float dcarry = 0.f;  // sums of the diagonals below the last block's, in lanes 0 .. 31
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 31, lh = lane >> 5;
  int b = a.remap ? xcd_block(blockIdx.x, gridDim.x) : static_cast<int>(blockIdx.x);
  const int pi = b % a.nparts;
  b /= a.nparts;
  const int tile = a.tiles - 1 - b % a.tiles;  // (under a causal mask the last rows see the most keys)
  b /= a.tiles;
  const int pass = b % a.passes, bh = b / a.passes, h = bh % a.H;
  if (MODE > 0 && a.flag[a.BH] != 0u && a.flag[bh] != 0u) return;  // (bwd_exact.hip)
  const int n = a.n, row0 = tile * kRows, wrow0 = row0 + 32 * wave;
  const int2 br = head_range(a.crange + static_cast<size_t>(h) * ctab_chunks(n), ctab_chunks(n), lane);
  int b0, b1, wlo = 0, whi = 0;
  key_blocks(br, n, row0, min(row0 + kRows, n) - 1, b0, b1);
  if (wrow0 < n) key_blocks(br, n, wrow0, min(wrow0 + 32, n) - 1, wlo, whi);
  {
    const int nb = b1 - b0, s = b0;
    b0 = s + static_cast<int>(static_cast<long long>(nb) * pi / a.nparts);
    b1 = s + static_cast<int>(static_cast<long long>(nb) * (pi + 1) / a.nparts);
  }
  // this wave's rows
  const size_t hb = static_cast<size_t>(bh) * a.nblk, xblk = hb + min(wrow0 >> 5, a.nblk - 1);
  uint4 x[KS][2];
  {
    const uint4* __restrict__ xp = a.X + xblk * NY * kFragLanes + lane;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int s = 0; s < 2; ++s) x[ks][s] = xp[(ks * 2 + s) * kFragLanes];
    keep(x);
  }
  uint4 x2[MODE == 2 ? KS2 : 1][2];
  int rp2 = 0;  // power of S2 S of this lane's row
  if constexpr (MODE == 2) {
    const uint4* __restrict__ xp = a.X2 + xblk * NY2 * kFragLanes + lane;
#pragma unroll
    for (int ks = 0; ks < KS2; ++ks)
#pragma unroll
      for (int s = 0; s < 2; ++s) x2[ks][s] = xp[(ks * 2 + s) * kFragLanes];
    keep(x2);
    rp2 = a.rpow[xblk * kBlk + lr] + a.rpow2[xblk * kBlk + lr];
    for (int e = lane; e < 64 * kDS; e += 64) diag[wave][e] = 0.f;
  }
  const uint32_t zbytes = static_cast<uint32_t>(a.ct_total) * 2 * NSZ * 1024u;  // per key block
  const int stride = ctab_stride(n);
  const __amdgpu_buffer_rsrc_t ry = buffer_of(a.Y + hb * NY * kFragLanes, static_cast<size_t>(a.nblk) * NY * 1024);
  const __amdgpu_buffer_rsrc_t ry2 = buffer_of(MODE == 2 ? a.Y2 + hb * NY2 * kFragLanes : a.Y,
                                               static_cast<size_t>(a.nblk) * NY2 * 1024);
  const __amdgpu_buffer_rsrc_t rz =
      buffer_of(reinterpret_cast<const char*>(a.Z) + hb * zbytes, static_cast<size_t>(a.nblk) * zbytes);
  const __amdgpu_buffer_rsrc_t rc = buffer_of(a.ctab + static_cast<size_t>(h) * stride, static_cast<size_t>(stride) * 4);
  const __amdgpu_buffer_rsrc_t rr = buffer_of(a.krec + hb * kRecWords, static_cast<size_t>(a.nblk) * kRecWords * 4);
  const __amdgpu_buffer_rsrc_t rr2 =
      buffer_of(MODE == 2 ? a.krec2 + hb * kRecWords : a.krec, static_cast<size_t>(a.nblk) * kRecWords * 4);
  const uint32_t lds0 = lds_address(&tiles_lds[0][0]), str0 = lds_address(&strip[0][0]);
  const uint32_t zpass = static_cast<uint32_t>(pass * CT * 2 * NSZ) * 1024u;
  // pieces of block blk into buffer `buf`: wave w stages pieces w, w + NW, ..:
  // the fragments, the c entries from key 32 blk and row row0 + kRows - 1 on,
  // the records
  auto stage = [&](int blk, int buf) {
    const uint32_t base = lds0 + static_cast<uint32_t>(buf) * (NF * 1024u), v16 = lane * 16u;
    const uint32_t sb = str0 + static_cast<uint32_t>(buf) * (kStrip * 4u);
    const uint32_t yo = static_cast<uint32_t>(blk) * (NY * 1024u), zo = static_cast<uint32_t>(blk) * zbytes + zpass;
    const uint32_t y2o = static_cast<uint32_t>(blk) * (NY2 * 1024u);
    const uint32_t co = static_cast<uint32_t>(32 * blk - row0 - (kRows - 1) + n - 1 + kCPad) * 4u;
    const uint32_t ro = static_cast<uint32_t>(blk) * (kRecWords * 4u);
    constexpr_for<(NF + NC + NR + NW - 1) / NW>([&](auto ic) {
      constexpr int lo = NW * decltype(ic)::value, hi = lo + NW - 1;  // this round's pieces
      const int f = lo + wave;
      if constexpr (hi < NY) {
        stage_lds<16>(ry, base + f * 1024u, v16, yo + f * 1024u);
      } else if constexpr (lo >= NY && hi < NY + NY2) {
        stage_lds<16>(ry2, base + f * 1024u, v16, y2o + (f - NY) * 1024u);
      } else if constexpr (lo >= NY + NY2 && hi < NF) {
        stage_lds<16>(rz, base + f * 1024u, v16, zo + (f - NY - NY2) * 1024u);
      } else {
        if (f < NY)
          stage_lds<16>(ry, base + f * 1024u, v16, yo + f * 1024u);
        else if (f < NY + NY2)
          stage_lds<16>(ry2, base + f * 1024u, v16, y2o + (f - NY) * 1024u);
        else if (f < NF)
          stage_lds<16>(rz, base + f * 1024u, v16, zo + (f - NY - NY2) * 1024u);
        else if (f < NF + NC)
          stage_lds<4>(rc, sb + (f - NF) * 256u, lane * 4u, co + (f - NF) * 256u);
        else if (f == NF + NC)
          stage_lds<4>(rr, sb + NC * 256u, lane * 4u, ro);
        else if (MODE == 2 && f == NF + NC + 1)
          stage_lds<4>(rr2, sb + (NC + 1) * 256u, lane * 4u, ro);
      }
    });
  };
  if (MODE == 0 && tid == 0) redo = 0u;
  Total zt[CT][16];
  double dsum = 0.0, wsum = 0.0;
  int kmost = -1000, vmost = -1000;  // largest powers of the keys and of the values
#pragma unroll
  for (int t = 0; t < CT; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) zt[t][e] = 0;
  if (b0 < b1) stage(b0, 0);
  for (int blk = b0; blk < b1; ++blk) {
    const int buf = (blk - b0) & 1;
    // this block's pieces are in LDS, the other buffer is consumed
    stage_wait();
    __syncthreads();
    if (blk + 1 < b1) stage(blk + 1, buf ^ 1);
    if (blk < wlo || blk >= whi) continue;
    const uint4* __restrict__ y = &tiles_lds[buf][lane];
    const uint4* __restrict__ zf = y + (NY + NY2) * kFragLanes;
    const float* __restrict__ rec = &strip[buf][NC * 64];
    const float* __restrict__ cs = &strip[buf][kRows - 1 - 32 * wave - lr + 4 * lh];
    floatx16 s, s1;
    s_product<KS>(y, x, s, s1);
    constexpr bool kAhead = KS <= kAheadSteps;
    float c16[kAhead ? 16 : 1], k16[kAhead ? 16 : 1];
    if constexpr (kAhead) {
      // read with the products: the table's entries and the record
#pragma unroll
      for (int e = 0; e < 16; ++e) c16[e] = cs[8 * (e >> 2) + (e & 3)];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 kr = *reinterpret_cast<const float4*>(rec + 8 * g + 4 * lh);
        k16[4 * g] = kr.x, k16[4 * g + 1] = kr.y, k16[4 * g + 2] = kr.z, k16[4 * g + 3] = kr.w;
      }
      s_schedule<KS>();
    }
    const int kexp = __builtin_amdgcn_readfirstlane(__float_as_int(rec[kRecE]));
    const int vexp = __builtin_amdgcn_readfirstlane(__float_as_int(rec[kRecV]));
    // P: lane row lr, keys 8 (e / 4) + 4 lh + e % 4
    float p[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) p[e] = fmaf(s1[e], kLoInv, s[e]);
    // w4: sums of the weights of S in P (they wait for no product)
    float w4[4] = {0.f, 0.f, 0.f, 0.f};
    if constexpr (kAhead) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        if (MODE == 0) w4[e & 3] = fmaf(k16[e], c16[e], w4[e & 3]);
        p[e] *= k16[e];
      }
    } else {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 kr = *reinterpret_cast<const float4*>(rec + 8 * g + 4 * lh);
        const float k4[4] = {kr.x, kr.y, kr.z, kr.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) p[4 * g + j] *= k4[j];
      }
    }
    if constexpr (MODE == 2) if (pass == 0) {  // uniform
      // the products (X2 Y2^T) o (X Y^T) of this block summed along its
      // diagonals: entry (key) of diagonal 32 + row - key, one diagonal per
      // lane to sum (slots that hold no entry stay zero; LDS float atomics
      // into one word per diagonal took four times as long as the rest of
      // the block).  Diagonals 32 .. 63 are complete after this block, the
      // next one's lie 32 below.
      const float* __restrict__ rec2 = rec + kRecWords;
      const uint4* __restrict__ y2 = y + NY * kFragLanes;
      floatx16 r, r1;
      s_product<KS2>(y2, x2, r, r1);
      const float f = ldexpf(1.f, rp2 + kexp + __float_as_int(rec2[kRecE]));
      float* __restrict__ win = &diag[wave][(32 + lr - 4 * lh) * kDS + 4 * lh];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 kr = *reinterpret_cast<const float4*>(rec2 + 8 * g + 4 * lh);
        const float k4[4] = {kr.x, kr.y, kr.z, kr.w};
#pragma unroll
        for (int j = 0; j < 4; ++j)
          win[(8 * g + j) * (1 - kDS)] = fmaf(r1[4 * g + j], kLoInv, r[4 * g + j]) * k4[j] * p[4 * g + j] * f;
      }
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      const float* __restrict__ dl = &diag[wave][lane * kDS];
      float up = __shfl(dcarry, lr);  // (lanes 32 .. 63 take the carry of 0 .. 31)
      up = lh == 1 ? up : 0.f;
#pragma unroll
      for (int k = 0; k < 32; ++k) up += dl[k];
      if (lh == 1) a.pdc[((hb + (wrow0 >> 5)) * (a.nblk + 1) + blk) * 32 + lr] = up;
      dcarry = up;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) p[e] *= kAhead ? c16[kAhead ? e : 0] : cs[8 * (e >> 2) + (e & 3)];
    if (32 * blk + 32 > n) {  // uniform: keys past n (of no weight, but c may be infinite)
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (32 * blk + 8 * (e >> 2) + 4 * lh + (e & 3) >= n) p[e] = 0.f;
    }
    float ds = 0.f, mx = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      if (MODE == 0) ds += p[e];
      mx = fmaxf(mx, fabsf(p[e]));
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    // the row's power in this block: its largest P is brought to [2^14, 2^15)
    // (zero and NaN maxima: 2^15, any power serves)
    const int ex = max(__builtin_amdgcn_frexp_expf(mx), -100) - 15;
    const float sc = __int_as_float((127 - ex) << 23);
    const int zexp = kexp + vexp + ex;
    Total zs;
    if constexpr (MODE == 0) {
      zs = exp2_int(zexp);
      dsum = fma(static_cast<double>(ds), exp2_int(kexp), dsum);
      if constexpr (!kAhead) {
        // (apart from P, whose registers it would take: it spills)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float4 kr = *reinterpret_cast<const float4*>(rec + 8 * g + 4 * lh);
          const float k4[4] = {kr.x, kr.y, kr.z, kr.w};
#pragma unroll
          for (int j = 0; j < 4; ++j) w4[0] = fmaf(k4[j], cs[8 * g + j], w4[0]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      const double ws = static_cast<double>((w4[0] + w4[1]) + (w4[2] + w4[3])) * exp2_int(kexp);
      wsum += ws;
      kmost = max(kmost, kexp);
      vmost = max(vmost, vexp);
    } else {
      zs = ldexpf(1.f, zexp);
    }
    uint4 ph[2], pl[2];
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2) {
      float v8[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) v8[t] = p[8 * k2 + t] * sc;
      split_f16x8(v8, kPLow, ph[k2], pl[k2]);
    }
#pragma unroll
    for (int t = 0; t < CT; ++t) {
      floatx16 zc = zero16(), z1 = zero16();
#pragma unroll
      for (int k2 = 0; k2 < 2; ++k2) {
        const uint4 vh = zf[((t * 2 + k2) * NSZ + 0) * kFragLanes];
        if constexpr (MODE > 0)
          z1 = mfma_f16(vh, pl[k2], z1);
        else
          zc = mfma_f16(vh, pl[k2], zc);
        zc = mfma_f16(vh, ph[k2], zc);
        if constexpr (NSZ > 1) z1 = mfma_f16(zf[((t * 2 + k2) * NSZ + 1) * kFragLanes], ph[k2], z1);
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const float zz = NSZ > 1 ? fmaf(z1[e], kLoInv, zc[e]) : zc[e];
        zt[t][e] = fma(static_cast<Total>(zz), zs, zt[t][e]);
      }
    }
  }
  const int i = wrow0 + lr;
  if constexpr (MODE == 0) {
    // a lane's sums cover this half-wave's keys, its columns those of its half
    dsum += __shfl_xor(dsum, 32);
    wsum += __shfl_xor(wsum, 32);
    // The test with every S taken as doubtful and a few columns ...
    // (Trigonometric features are as large as their position's amplitude allows
    // and S cancels: its size does not say that a term was not held, nor the
    // denominator how large P's entries are.)
    const bool trf = a.kind == kFeatTrf;
    const double beside = kUnderflow * exp2_int(kmost + 11);  // (2^11 blocks at most)
    const double off = fma(trf ? 0.0 : kDoubtErr<KS>, wsum, beside), mass = trf ? wsum * (16.0 * KS * 0x1p30) : dsum;
    const double offn = fma(kSplitFloor, mass, off) * exp2_int(vmost + 15);
    double num = fmax(fmax(fabs(zt[0][0]), fabs(zt[0][1])), fmax(fabs(zt[0][2]), fabs(zt[0][3])));
    bool again = false;
    if (__builtin_expect(__any(i < n && !(off <= kRowTau * fabs(dsum) && offn <= kRowTau * num)), 0)) {
      // ... and in full, where that does not pass
#pragma unroll
      for (int t = 0; t < CT; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) num = fmax(num, fabs(zt[t][e]));
      num = fmax(num, __shfl_xor(num, 32));
      again = !rows_held<KS>(a, bh, wrow0, max(b0, wlo), min(b1, whi), dsum, num, wsum, beside, vmost);
    }
    if (__builtin_expect(again, 0)) {
      if (lane == 0) atomicOr(&redo, 1u << wave);
    } else if (wrow0 < n) {
      store_rows<CT, NW>(a, bh, pass, tile, pi, wave, zt, dsum);
    }
    __syncthreads();
    if (__builtin_expect(redo != 0u, 0)) {
      // (the arguments are read anew: none is held through the loop above for this)
      const DirectArgs* ap = (const DirectArgs*)__builtin_amdgcn_kernarg_segment_ptr();
      asm volatile("" : "+s"(ap));
      if (ap->flag && tid == 0) ap->flag[bh] = ap->flag[ap->BH] = 1u;
      const unsigned mask = __builtin_amdgcn_readfirstlane(redo);
#pragma unroll 1
      for (int w = 0; w < NW; ++w) {
        if ((mask >> w & 1u) == 0u) continue;
        exact_rows<TV, KS, CT, NW>(*ap, reinterpret_cast<float4*>(&tiles_lds[0][0]), den, bh, pass, tile, pi, w, b0,
                                   b1);
        if (wave == w) dsum = den[lr];
      }
    }
  }
  if (wrow0 >= n) return;  // uniform per wave; no barrier follows
  if constexpr (MODE > 0) {
    const float rs = ldexpf(1.f, a.rpow[xblk * kBlk + lr]);
    if (MODE == 2 && pass == 0 && lh == 0 && whi > wlo)  // the diagonals below the last block's
      a.pdc[((hb + (wrow0 >> 5)) * (a.nblk + 1) + whi) * 32 + lr] = dcarry;
    if (a.ldz == 0) {
      float4* __restrict__ o = reinterpret_cast<float4*>(a.z) + (xblk * a.out_ks * kFragLanes + lane) * 2;
#pragma unroll
      for (int t = 0; t < CT; ++t)
#pragma unroll
        for (int k2 = 0; k2 < 2; ++k2) {
          const int ks = 2 * (pass * CT + t) + k2;
          if (ks >= a.out_ks) continue;  // uniform
          const Total* __restrict__ q = &zt[t][8 * k2];
          o[ks * 2 * kFragLanes] = make_float4(q[0] * rs, q[1] * rs, q[2] * rs, q[3] * rs);
          o[ks * 2 * kFragLanes + 1] = make_float4(q[4] * rs, q[5] * rs, q[6] * rs, q[7] * rs);
        }
    } else if (i < n) {
      float* __restrict__ zr = a.z + (static_cast<size_t>(bh) * n + i) * a.ldz;
#pragma unroll
      for (int t = 0; t < CT; ++t)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int c = (pass * CT + t) * 32 + 8 * g + 4 * lh;
          const Total* __restrict__ q = &zt[t][4 * g];
          store4(zr, c, a.ldz, q[0] * rs, q[1] * rs, q[2] * rs, q[3] * rs);
        }
    }
  } else {
    double* __restrict__ part = part_of<CT, NW>(a, bh, pass, tile, pi) + 32 * wave + lr;  // [column][row]
    float* __restrict__ zr = a.z + (static_cast<size_t>(bh) * n + i) * a.d;
    // Values that are not finite and those too small for their block's power
    // (rows evaluated again have these), stored as zeros, their blocks flagged:
    // P v added in fp64, one key at a time; rare.
    const unsigned* __restrict__ vf = a.vflag + hb;
    const int f0 = max(b0, wlo), f1 = min(b1, whi);
    const unsigned kinds = (redo >> wave & 1u) != 0u ? 1u : 3u;
    bool odd = false;
    for (int blk = f0 + lane; blk < f1; blk += 64) odd |= (vf[blk] & kinds) != 0u;
    if (!__any(odd)) return;
    __threadfence();  // the rows stored above are read back below, by other lanes
    const TV* __restrict__ v = static_cast<const TV*>(a.v) + static_cast<size_t>(bh) * n * a.d;
    const float* __restrict__ ct = a.ctab + static_cast<size_t>(h) * stride + kCPad + n - 1;
    const int cbeg = pass * CT * 32, cend = min(a.d, cbeg + CT * 32);
    auto value = [](uint4 hh, uint4 ll, int j) {  // element j of a pair of fragments
      const uint32_t w[4] = {hh.x, hh.y, hh.z, hh.w}, u[4] = {ll.x, ll.y, ll.z, ll.w};
      return term_value(w[j >> 1], u[j >> 1], j & 1);
    };
    for (int blk = f0; blk < f1; ++blk) {
      if ((vf[blk] & kinds) == 0u) continue;
      const float* __restrict__ rec = a.krec + (hb + blk) * kRecWords;
      const int vexp = __float_as_int(rec[kRecV]);
      auto missing = [&](int key, int c) {  // what the sums lack of v[key][c]
        const float x1 = to_f32(v[static_cast<size_t>(key) * a.d + c]);
        if (!isfinite(x1)) return x1;
        return kinds == 1u ? 0.f : ldexpf(apart<NSZ>(ldexpf(x1, -vexp)), vexp);
      };
      for (int key = 32 * blk; key < min(32 * blk + 32, n); ++key) {
        bool any = false;
        for (int c = cbeg + lane; c < cend; c += 64) any |= missing(key, c) != 0.f;
        if (!__any(any)) continue;
        // S of (row, key): this lane half's slots, then the other half's
        float s = 0.f;
        const uint4* __restrict__ yp = a.Y + (hb + blk) * NY * kFragLanes + 32 * lh + (key & 31);
        const uint4* __restrict__ xp = a.X + xblk * NY * kFragLanes + lane;
#pragma unroll 2
        for (int ks = 0; ks < KS; ++ks) {
          const uint4 xh = xp[(ks * 2 + 0) * kFragLanes], xl = xp[(ks * 2 + 1) * kFragLanes];
          const uint4 yh = yp[(ks * 2 + 0) * kFragLanes], yl = yp[(ks * 2 + 1) * kFragLanes];
#pragma unroll
          for (int j = 0; j < 8; ++j) s = fmaf(value(xh, xl, j), value(yh, yl, j), s);
        }
        s += __shfl_xor(s, 32);
        if (lh != 0 || i >= n || ct[key - i] == 0.f) continue;  // (a masked key reaches no row)
        const double p = static_cast<double>(s * rec[key & 31] * ct[key - i]) * exp2_int(__float_as_int(rec[kRecE]));
        for (int c = cbeg; c < cend; ++c) {
          const float x1 = missing(key, c);
          if (x1 == 0.f) continue;
          if (a.nparts == 1)
            zr[c] = static_cast<float>(zr[c] + p * x1 / dsum);
          else
            part[(c - cbeg) * kRows] += p * x1;
        }
      }
    }
  }
}

}  // namespace krpe
