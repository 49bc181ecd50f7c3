// Weighted products on the fp16 matrix cores, at fp32 accuracy.
//
// Eq. (10) evaluated directly has the form
//
//   out_r = sum_j ((X Y^T)_rj c_{j-r}) Z_j
//
// with X, Y (phi(q), phi(k)) contracted over features and Z (v) over
// positions.  Every fp32 operand is held as a power of two and two fp16 terms,
//
//   a = 2^e (h + 2^-11 l),   h = fp16(2^-e a),  l = fp16(2^11 (2^-e a - h)),
//
// e from the largest |a| that shares the power (the features of one position;
// the block of 32 positions for Z), which is brought to [2^14, 2^15).  The two
// terms represent 2^-e a to 2^-23 of itself down to 2^-13, 28 binades below
// that largest element, and to an absolute 2^-36 below.  So an S whose terms
// all pair one position's largest features with the other's smallest (keys that
// oppose the query, norms well above d^(1/4)) is not held; the forward pass
// bounds what each row may have lost that way and evaluates the rows that do not
// pass in fp32 from q, k and W (direct_args.hpp, direct_exact.hpp).  A product takes the
// three terms h h, h l and l h (l l is below 2^-22 of it): three fp16 MFMAs of
// 16 contraction steps, 32 cycles each, against eight fp32 MFMAs of two, 64
// cycles each, 5.3 times the fp32 matrix rate.  Products are exact and sums
// are fp32 in the MFMA; h h and the two small products run in accumulators of
// their own, so the small ones do not cost roundings of the large sum.
//
// Fragments.  An operand is stored as the MFMA reads it: fragments of 64 lanes
// x 8 fp16 (1 KiB), so that a tile is a run of whole fragments, copied to LDS
// by 16-byte-per-lane direct loads and read back conflict-free.  With lane =
// 32 lh + lr and slot t < 8:
//   S operands (X, Y; [block][k step][term]): position 32 block + lr, feature
//     16 ks + 8 (t / 4) + 4 lh + t % 4;
//   Z operands ([block][column tile][k step < 2][term]): column 32 ct + lr,
//     position 32 block + 16 k2 + 8 (t / 4) + 4 lh + t % 4.
// The order within a k step is the one in which a 32 x 32 MFMA result leaves
// its rows in a lane (register e of lane half lh holds row 8 (e / 4) + 4 lh +
// e % 4): the feature map writes S fragments from its accumulators, and the
// weights P leave the first product as an operand of the second, without any
// exchange between lanes.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "common.hpp"

namespace krpe {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kBlk = 32;        // positions per fragment block
constexpr int kFragLanes = 64;  // uint4 per fragment
// The table of c = exp(b): kCPad zeros, c_t for t = -(n-1) .. n-1, zeros to
// the end, so that every entry a tile of up to 256 rows reads lies inside it.
constexpr int kCPad = 384;
constexpr int kCChunk = 2048;  // table entries per work-group of the table's kernel
__host__ __device__ constexpr int ctab_stride(int n) { return (2 * n - 1 + 2 * kCPad + 63) & ~63; }
__host__ __device__ constexpr int ctab_chunks(int n) { return (ctab_stride(n) + kCChunk - 1) / kCChunk; }

// ---- bf16 terms of fp32 values, a = a_0 + a_1 + a_2 exactly (the projections
// of the feature map, whose operands come unscaled)
__device__ __forceinline__ uint32_t pack_bf16(floatx2 v) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ floatx2 minus_bf16(floatx2 v, uint32_t h) {
  v.x -= __uint_as_float(h << 16);
  v.y -= __uint_as_float(h & 0xffff0000u);
  return v;
}
__device__ __forceinline__ void split_bf16(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l) {
  floatx2 v;
  v.x = a;
  v.y = b;
  h = pack_bf16(v);
  v = minus_bf16(v, h);
  m = pack_bf16(v);
  v = minus_bf16(v, m);
  l = pack_bf16(v);
}
__device__ __forceinline__ void split_bf16x8(const float (&x)[8], uint4 (&t)[3]) {
  split_bf16(x[0], x[1], t[0].x, t[1].x, t[2].x);
  split_bf16(x[2], x[3], t[0].y, t[1].y, t[2].y);
  split_bf16(x[4], x[5], t[0].z, t[1].z, t[2].z);
  split_bf16(x[6], x[7], t[0].w, t[1].w, t[2].w);
}
__device__ __forceinline__ floatx16 mfma_bf16(uint4 a, uint4 b, floatx16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                 0, 0);
}

// ---- fp16 terms
constexpr float kLoScale = 2048.f, kLoInv = 1.f / 2048.f;  // 2^11
__device__ __forceinline__ uint32_t pack_f16(float a, float b) {
  floatx2 v;
  v.x = a;
  v.y = b;
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, halfx2));
}
// a - fp16 half of h (exact), one instruction (the compiler converts and
// subtracts)
__device__ __forceinline__ float minus_f16_lo(float a, uint32_t h) {
  float r;
  asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(r) : "v"(h), "v"(a));
  return r;
}
__device__ __forceinline__ float minus_f16_hi(float a, uint32_t h) {
  float r;
  asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(h), "v"(a));
  return r;
}
// (a, b) = h + l / lo, lo = 1 or kLoScale
__device__ __forceinline__ void split_f16(float a, float b, float lo, uint32_t& h, uint32_t& l) {
  h = pack_f16(a, b);
  l = pack_f16(minus_f16_lo(a, h) * lo, minus_f16_hi(b, h) * lo);
}
__device__ __forceinline__ void split_f16x8(const float (&x)[8], float lo, uint4& h, uint4& l) {
  split_f16(x[0], x[1], lo, h.x, l.x);
  split_f16(x[2], x[3], lo, h.y, l.y);
  split_f16(x[4], x[5], lo, h.z, l.z);
  split_f16(x[6], x[7], lo, h.w, l.w);
}
// An element of Z too small for its power's terms (the power's largest is 2^31 or
// more above it) is not split but added apart, else zero.  TERMS = 2: above 2^-16
// the terms hold it, and the product l l that is dropped, to 2^-20 of it; 1 (bf16
// values): above 2^-17 it is an fp16 number.
template <int TERMS>
__device__ __forceinline__ float apart(float a) {
  return fabsf(a) < (TERMS == 2 ? 0x1p-16f : 0x1p-17f) ? a : 0.f;
}
// the value of half j (0, 1) of a pair of terms, l scaled by kLoScale
__device__ __forceinline__ float term_value(uint32_t h, uint32_t l, int j) {
  const halfx2 hp = __builtin_bit_cast(halfx2, h), lp = __builtin_bit_cast(halfx2, l);
  return fmaf(static_cast<float>(j ? lp.y : lp.x), kLoInv, static_cast<float>(j ? hp.y : hp.x));
}
__device__ __forceinline__ floatx16 mfma_f16(uint4 a, uint4 b, floatx16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(halfx8, a), __builtin_bit_cast(halfx8, b), c, 0, 0,
                                                0);
}
__device__ __forceinline__ floatx16 zero16() {
  floatx16 z;
#pragma unroll
  for (int e = 0; e < 16; ++e) z[e] = 0.f;
  return z;
}
// 2^e as a double, |e| < 1023
__device__ __forceinline__ double exp2_int(int e) {
  return __longlong_as_double(static_cast<long long>(1023 + e) << 52);
}

// Copies `bytes` per lane (4 or 16) from the buffer at lane offset voff plus
// the uniform offset soff to LDS at the uniform byte address `lds` + lane x
// bytes, without passing through registers.  Completion counts in vmcnt only:
// stage_wait() before the barrier that publishes the data.
template <int BYTES>
__device__ __forceinline__ void stage_lds(__amdgpu_buffer_rsrc_t r, uint32_t lds, uint32_t voff, uint32_t soff) {
  static_assert(BYTES == 4 || BYTES == 16, "stage_lds: 4 or 16 bytes per lane");
  // m0 holds the LDS address (one wait state between its write and the load);
  // the wait states also cover an SGPR operand that a VALU instruction (a
  // readfirstlane) has just written, five before a vector memory instruction
  // reads it: the compiler does not look into the statement for that.
  if constexpr (BYTES == 16)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds), "v"(voff),
                 "s"(r), "s"(soff)
                 : "memory");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dword %1, %2, %3 offen lds" ::"s"(lds), "v"(voff), "s"(r),
                 "s"(soff)
                 : "memory");
}
__device__ __forceinline__ void stage_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const char*)p));
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0,
                                           static_cast<int>(bytes < 0x7fffffffu ? bytes : 0x7fffffffu), 0x00020000);
}

// Range [lo, hi] of s = t + n - 1 with c_t != 0 of one head, from the chunk
// ranges of its table; every lane of the wave receives it.
__device__ __forceinline__ int2 head_range(const int2* __restrict__ chunk_range, int chunks, int lane) {
  int lo = 1 << 30, hi = -1;
  for (int c = lane; c < chunks; c += 64) {
    lo = min(lo, chunk_range[c].x);
    hi = max(hi, chunk_range[c].y);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    lo = min(lo, __shfl_xor(lo, off));
    hi = max(hi, __shfl_xor(hi, off));
  }
  return make_int2(__builtin_amdgcn_readfirstlane(lo), __builtin_amdgcn_readfirstlane(hi));
}

}  // namespace krpe
