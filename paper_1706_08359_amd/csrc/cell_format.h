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

#endif  // GBDT_CELL_FORMAT_H_
