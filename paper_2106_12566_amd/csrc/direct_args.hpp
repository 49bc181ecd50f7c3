// Records and arguments of the weighted products' kernel (direct_kernel.hpp).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace krpe {

// Record of a 32-key block, 64 words: [0, 32) 2^(e_j - E) per key, e_j the
// power of phi(k_j) and E = word 32 (int); word 33 (int) the power of its
// values; word 34 the largest sum of a key's features in units of its power
// (PRF and elu + 1).
constexpr int kRecWords = 64, kRecE = 32, kRecV = 33, kRecSum = 34;
// S of two positions is at most 2^30 M in units of their powers: E carries 30
// of them, so that P stays near c_{j-i}'s range.
constexpr int kRecBias = 30;
// Rows of the forward pass that two fp16 terms do not hold (wprod.hpp).  A term is
// off by at most 2^-36 of its position's unit where it does not hold its feature
// to 2^-23, and the product l l of such a term by 2^-37 of that unit times the
// other's, so an S by less than kTermErr times the sums of both positions' features,
// 16 KS 2^15 each at most (kDoubtErr; a few 2^15 where S can be small, as one
// feature then exceeds the others by far).  An S below kDoubt times that is doubtful.
// A row is held if what its doubtful entries may be off by, weighted as in the
// sums, is at most kRowTau of its denominator and, with their values, of its
// largest numerator.
// Two more losses count: kUnderflow, in units of the block's power, for each entry
// whose weight may have left fp32's range (b near the range's end, a key far below
// one of its block that the row does not see), and kSplitFloor of the block's
// largest entry, below which P's terms lose its others, with its largest value.
// k_direct tests this with every entry taken as doubtful and the largest sums
// (inputs scaled by d^(-1/4) pass by 2^8 and more), rows_held with the sums, then
// in full, and exact_rows evaluates the rows of a wave that fails.
constexpr double kRowTau = 0x1p-20, kTermErr = 0x1p-35, kDoubt = 0x1p21;
template <int KS>
constexpr double kDoubtErr = kTermErr * 2 * 16 * KS * 32768.0;
constexpr double kUnderflow = 0x1p-111, kSplitFloor = 0x1p-36;

struct DirectArgs {
  const uint4 *X, *Y, *Z;
  const float* krec;
  const unsigned* vflag;
  const float* ctab;
  const int2* crange;
  const void* v;
  float* z;
  double* den;       // denominators in units of the queries' powers (or NULL)
  const int* rpow;   // MODE 1, 2: powers of the rows [BH][32 nblk]
  int ldz;           // MODE 1, 2: row length of z; 0: z as fp32 S fragments of out_ks k steps
  int out_ks;
  const uint4 *X2, *Y2;  // MODE 2: the second pair of operands ([block][KS2][2])
  const float* krec2;    // its keys' records
  const int* rpow2;      // and rows' powers
  float* pdc;            // diagonal sums [BH][nblk row blocks][32 (nblk + 1)]
  double* part;
  int BH, H, n, nblk, d, ct_total, tiles, passes, nparts, remap;
  // MODE 0: what a row tile is evaluated from in fp32 (direct_exact.hpp)
  const void *q, *k;
  const float* W;
  const int* qpow;  // powers of phi(q) [BH][32 nblk]
  const float* qsum;  // and sums in their units
  unsigned* flag;   // [BH + 1] heads with such a tile; any head (written, MODE 1, 2: these heads are skipped)
  int m, kind, nprf;
  float inv_sqrt_m;
  double log2_m;
};

}  // namespace krpe
