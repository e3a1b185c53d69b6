// The 64-bit cell in which a workgroup of the build kernels counts and sums the rows of one (bin,
// feature) pair over an epoch.  Shared by the kernels and by the host (tests).
#ifndef GBDT_CELL_FORMAT_H_
#define GBDT_CELL_FORMAT_H_

#include <stdint.h>

#include "tile_plan.h"

// A histogram cell is ONE 64-bit integer that carries, from the low bits up, the
// count (10 bits), the quantised gradient sum (27 bits, signed) and the quantised
// hessian sum (27 bits, signed).  A workgroup drains its cells after every epoch
// of kEpochRows rows, so a cell receives at most 512 additions between drains.
// (Wide cells of 256 bins may be drained once in two epochs: see below.)
//
// The count lies below the sums because it has to be exact whatever they do: nothing that overflows
// above can reach it, neither the sums of finite values whose sum of magnitudes is past the largest
// fp32 number (no scale keeps those inside 27 bits) nor what a conversion makes of an infinity.  Tree growth
// finds the rows of a node by its counts, so a wrong count would be an address out of range.  (With the
// gradient sum in the lowest bits, under a bias, a drained cell takes 9 vector instructions instead of 10,
// but its overflow runs into the count.)
constexpr int kEpochRows = 512;
constexpr int kCountBits = 10;
constexpr int kSumBits = 27;
static_assert(kEpochRows < (1 << kCountBits), "an epoch's count must fit its field");
static_assert(kCountBits + 2 * kSumBits == 64, "the three fields fill the cell");
constexpr int kSumPad = 32 - kSumBits;  // a sum in the upper bits of a signed word is 2^kSumPad times itself

// What a row adds to its cells: 1 + gq * 2^10 + hq * 2^37 (two's complement).
struct CellWords {
  uint32_t lo, hi;
};
GBDT_HD CellWords cell_addend(int32_t gq, int32_t hq) {
  CellWords w;
  w.lo = ((uint32_t)gq << kCountBits) + 1u;
  w.hi = (uint32_t)(gq >> (32 - kCountBits)) + ((uint32_t)hq << (kCountBits + kSumBits - 32));
  return w;
}

// The fields of a cell, the sums times 2^kSumPad: moved to the upper bits of a word each, a sum
// needs no sign extension.  The hessian sum sits above a borrow of one when the gradient sum is
// negative; adding half of its unit gives it back (bit 36, the gradient sum's sign, carries).
struct CellSums {
  int32_t grad, hess;
  uint32_t count;
};
GBDT_HD CellSums cell_sums(uint32_t lo, uint32_t hi) {
  constexpr uint32_t kTop = ~((1u << kSumPad) - 1u);
  CellSums s;
  s.grad = (int32_t)(((hi << (32 - kSumPad)) | (lo >> kSumPad)) & kTop);
  s.hess = (int32_t)((hi + (1u << (kSumPad - 1))) & kTop);
  s.count = lo & ((1u << kCountBits) - 1u);
  return s;
}
static_assert(kCountBits == 2 * kSumPad, "bits kCountBits and up of a cell are bits kSumPad and up of the word taken at kSumPad");

// Power-of-two scale 2^k for quantising the values of one epoch to integers: the
// largest k with 2^k * m + kEpochRows / 2 (rounding slack) < 2^26, so that no cell's
// signed 27-bit field can overflow whatever the bins are.  m_bits: the bit pattern of
// m = 1.002 * (fp32 sum of |v| over the epoch) (the factor covers the rounding of the
// sum itself).  Integer arithmetic only: on a wave-uniform value it runs on the
// scalar unit.  A zero (or denormal) sum gives k = 0; k is kept in [-126, 126] so
// that 2^k and 2^-k are normal floats.  (The drain's 2^-(k + kSumPad) is a denormal from k = 122 on,
// which the multiply-adds take as it is.)
GBDT_HD int epoch_scale_exp(uint32_t m_bits) {
  const int e = (int)((m_bits >> 23) & 0xffu);
  const uint32_t mant = m_bits & 0x7fffffu;
  if (e == 0) return 0;
  int k = (kSumBits - 2) + 127 - e;  // 2^k * m in [2^25, 2^26)
  // 2^k * m = (1 + mant / 2^23) * 2^25 > 2^26 - kEpochRows  <=>  mant > 2^23 - kEpochRows / 4
  if (mant > (1u << 23) - (uint32_t)(kEpochRows >> (kSumBits - 25))) k -= 1;
  if (k > 126) k = 126;
  if (k < -126) k = -126;
  return k;
}
// Wide accumulation (the double precision switch of App. A.6): a (bin, feature) pair owns TWO
// 64-bit cells, gradient and hessian, each a signed 54-bit sum above the 10-bit count field (the
// count is kept in the gradient cell).  Values are scaled by 2^(k + kWideShift), k the exponent
// of the narrow format, so an epoch's sum of magnitudes stays below 2^50 and a value is rounded
// at 2^-50 of it at worst -- a fp32 value that is not 2^26 times smaller than the epoch's sum is
// taken exactly.  Cells are drained into fp64 accumulators.  Twice the LDS atomics and twice the
// LDS space of the default format.
constexpr int kWideShift = 24;
// The 256-bin variants drain their cells once in two epochs (kPairs in build_tile) and scale by one more power of two: an epoch's
// sum of magnitudes stays below 2^51.  So does that of a second epoch, taken with the scale of the first, if its exponent is the same
// or one more; if it is one less, the sum, and a lone row of it, may come near 2^52.  Either way both together are below 2^53 and fit
// the field.
constexpr int kWideShiftOfTwo = 25;
GBDT_HD double pow2d(int k) { return __builtin_bit_cast(double, (long long)(k + 1023) << 52); }
// An epoch whose sum of magnitudes is past the largest fp32 number has no scale of its own: it is scaled as if the sum
// were 2^128, with this exponent (and kWideShift always).  The 54-bit field of a cell then takes fifteen rows of the largest number,
// which is more than the 2^51 that i64_to_f64 takes: epochs of this exponent are drained by a conversion of all 53 bits of a double.
constexpr int kWidePastExp = (kSumBits - 2) + 127 - 255;
GBDT_HD int wide_cell_exp(int k, bool pairs) { return k + (pairs && k > kWidePastExp ? kWideShiftOfTwo : kWideShift); }
// Whether the sums of an epoch of exponent k and of the next one, of exponent k2, fit the same cells at the scale of the first.
GBDT_HD bool wide_pair(int k, int k2) { return (uint32_t)(k - k2 + 1) <= 2u && k > kWidePastExp + 1; }
// round-to-nearest-even of |v| <= 2^51 to a 64-bit integer (the sum's low mantissa bits)
GBDT_HD long long rint_to_i64(double v) {
  return __builtin_bit_cast(long long, v + 6755399441055744.0) - 0x4338000000000000LL;
}
// A row's value at the scale 2^exp.  coarse: 0, or 1 for a second epoch whose own exponent is one less: its values go past what
// rint_to_i64 takes, so they are rounded at half the scale, which is the epoch's own, and doubled.
GBDT_HD long long wide_quantise(float v, int exp, int coarse) {
  return (long long)((unsigned long long)rint_to_i64((double)v * pow2d(exp - coarse)) << coarse);
}

#endif  // GBDT_CELL_FORMAT_H_
