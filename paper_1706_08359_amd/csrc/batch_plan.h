// Tables of a batched histogram launch (several leaves in one grid) and the mapping of a
// block of that grid to its work.  Shared by the kernel and by the host (planning, tests).
#ifndef GBDT_BATCH_PLAN_H_
#define GBDT_BATCH_PLAN_H_

#include <stdint.h>

#include "tile_plan.h"

constexpr int kBatchLeaves = 224;  // leaves per launch: the table travels as kernel arguments (4 KB at most)

struct BatchLeaf {
  uint32_t row_off;   // first entry of the leaf's row list
  uint32_t n;         // its length
  uint32_t first_wg;  // workgroups per tile of all earlier leaves of the table
  uint32_t packed;    // workgroups per tile | epochs per unit << 16 | number of the leaf in the call's launch << 24
};
GBDT_HD uint32_t batch_leaf_pack(uint32_t wgs, uint32_t unit_epochs, uint32_t leaf) {
  return wgs | (unit_epochs << 16) | (leaf << 24);
}
GBDT_HD uint32_t batch_wgs(const BatchLeaf& l) { return l.packed & 0xffffu; }
GBDT_HD uint32_t batch_unit_epochs(const BatchLeaf& l) { return (l.packed >> 16) & 0xffu; }
GBDT_HD uint32_t batch_leaf_no(const BatchLeaf& l) { return l.packed >> 24; }
static_assert(kBatchLeaves <= 256, "a leaf's number has 8 bits");

// Blocks of a launch with `cols` workgroup columns (one workgroup of every tile): block ->
// (tile, column).  Workgroups that read the same cache lines -- the tiles of one line of the
// matrix, same column and so the same rows at the same time -- are kept on one XCD, whose L2 then
// fetches the line once.  Consecutive blocks go to the 8 XCDs in turn, so eight (line, column)
// pairs are dealt out at a time and their tiles follow one another 8 blocks apart; the
// pairs left over (fewer than 8) come last.  Tiles that make no whole line follow, the remainder tile
// last of all unless it shares a region: its blocks have the least work, and where the grid does not fill
// the machine evenly they are what the last CUs should get (300,000 x 193 x 63, 588 blocks on 256 CUs:
// dealt out with the lone main tile's the root took 34.7 us, behind them 30.6).  In a batched launch pairs are numbered column after
// column, so that blocks start in the order of the columns, the longest first; a single leaf's blocks
// all start at once, and there a line's columns are numbered through, so that (with a multiple
// of 8 columns) the lines of a column, which read the same gradients and hessians, share an XCD too.
// Not so where a region has one tile, and where the workgroups take one epoch each (short leaves): nothing can run
// behind the other then and find its line there, both wait for the same one at the same time, and the
// tiles are better spread over the XCDs: 50,000 x 500 x 64, two leaves of half the rows together 21.5 us dealt
// by lines, 20.1 so; 30,000 x 1,000 x 64, half of the rows 21.1 and 19.9.  With two epochs each it is the other way round
// (30,000 x 1,000 x 64, all rows: 21.4 us dealt by lines, 24.4 so) unless the launch leaves CUs without a workgroup, as
// only those with one workgroup a CU do: latency counts there, not traffic (256 bins, wide accumulation, 172 blocks: 700,000 x
// 50, an eighth of the rows 20.3 us dealt by lines, 17.7 so; 144 blocks, 300,000 x 500, a 32nd 37.9 and 35.3).
constexpr uint32_t kXcds = 8;
// With wide accumulation a workgroup is as fast as its CU lets it, and one beside a workgroup of the remainder tile is faster.
// The hand-out of units evens that out within a tile, so every tile has to have workgroups on both kinds of CU: a lone main
// tile between the pairs and the remainder tile has them all where no remainder is.  There its blocks are dealt
// out with the pairs', eight columns at a time (tile after tile of them: pairs stay 8 blocks apart).  3,000,000 x 400 x 16,
// root 522 us behind the pairs, 479 so (467 with a region per tile); 1,500,000 x 330 x 64 238 and 222.  (Without wide
// accumulation memory evens the CUs out, and the order by lines is the better one: 11,000,000 x 700 x 16, root 1,410 us, 1,450
// so.)
enum DealOrder : int32_t { kDealTiles = 0, kDealLines = 1, kDealColumns = 2 };
GBDT_HD int32_t deal_order(int32_t line_tiles, int32_t unit_epochs, int64_t blocks, int32_t cus, bool wide) {
  if (line_tiles == 1 || unit_epochs < 2 || (unit_epochs == 2 && blocks < cus)) return kDealTiles;
  return wide ? kDealColumns : kDealLines;
}
struct LineBlock {
  int32_t tile;
  uint32_t col;
};
GBDT_HD void line_deal(uint32_t b, uint32_t n_pairs, uint32_t* pair, uint32_t* tile) {  // two tiles a line
  const uint32_t dealt = n_pairs / kXcds * kXcds;
  if (b < dealt * 2u) {
    const uint32_t i = b / kXcds;
    *pair = i / 2u * kXcds + b % kXcds;
    *tile = i % 2u;
  } else {
    const uint32_t r = b - dealt * 2u, rest = n_pairs - dealt;
    *tile = r < rest ? 0u : 1u;
    *pair = dealt + r - *tile * rest;
  }
}
GBDT_HD LineBlock line_block(int32_t wm, int32_t n_main, int32_t wr, int32_t deal, uint32_t cols, bool by_column,
                             uint32_t b) {
  LineBlock r;
  if (n_main + (wr ? 1 : 0) == 1) {
    r.tile = 0;
    r.col = b;
    return r;
  }
  if (deal == kDealTiles) {  // neighbouring blocks take different tiles
    const uint32_t main_blocks = (uint32_t)n_main * cols;
    r.tile = b < main_blocks ? (int32_t)(b % (uint32_t)n_main) : n_main;
    r.col = b < main_blocks ? b / (uint32_t)n_main : b - main_blocks;
    return r;
  }
  const uint32_t lines = (uint32_t)n_main / 2u;
  uint32_t pair = 0, tile = 0;
  if (deal == kDealColumns && (n_main & 1) && lines && !plan_leftover_shared(wm, n_main, wr)) {
    const uint32_t chunk = kXcds * (uint32_t)n_main, in_chunks = cols / kXcds * chunk;
    if (b < in_chunks) {
      const uint32_t k = b / chunk, i = b - k * chunk;
      r.tile = (int32_t)(i / kXcds);
      r.col = k * kXcds + i % kXcds;
      return r;
    }
    // the last few columns, as below
    LineBlock rest = {0, 0};
    const uint32_t n = cols % kXcds;
    b -= in_chunks;
    if (b < lines * n * 2u) {
      line_deal(b, lines * n, &pair, &tile);
      rest.tile = (int32_t)(pair % lines * 2u + tile);
      rest.col = pair / lines;
    } else if (b < (uint32_t)n_main * n) {
      rest.tile = n_main - 1;
      rest.col = b - lines * n * 2u;
    } else {  // the remainder tile, every column of it
      r.tile = n_main;
      r.col = b - (uint32_t)n_main * n;
      return r;
    }
    rest.col += cols - n;
    return rest;
  }
  const uint32_t line_blocks = lines * cols * 2u;
  if (b < line_blocks) {
    line_deal(b, lines * cols, &pair, &tile);
    const uint32_t per = by_column ? lines : cols;
    const uint32_t q = pair / per, rem = pair - q * per;
    r.tile = (int32_t)((by_column ? rem : q) * 2u + tile);
    r.col = by_column ? q : rem;
    return r;
  }
  b -= line_blocks;  // the tiles that make no whole line
  if (plan_leftover_shared(wm, n_main, wr)) {
    line_deal(b, cols, &pair, &tile);
  } else {
    tile = b < cols ? 0u : 1u;
    pair = b - tile * cols;
  }
  r.tile = (int32_t)(lines * 2u + tile);
  r.col = pair;
  return r;
}

// The same for a launch whose main tiles are built in halves (plan_halves): the two halves of a (tile, column) follow
// one another 8 blocks apart, as the tiles of a line do, because they read the same bytes; the remainder tile, which has no
// halves, comes last.
struct HalfBlock {
  int32_t tile, half;
  uint32_t col;
};
GBDT_HD HalfBlock half_block(int32_t wm, int32_t n_main, int32_t deal, uint32_t cols, bool by_column, uint32_t b) {
  const uint32_t main_blocks = (uint32_t)n_main * cols, dealt = main_blocks / kXcds * kXcds;
  HalfBlock r;
  if (b >= 2u * main_blocks) {
    r.tile = n_main;
    r.half = 0;
    r.col = b - 2u * main_blocks;
    return r;
  }
  uint32_t of;
  if (b < 2u * dealt) {
    const uint32_t i = b / kXcds;
    r.half = (int32_t)(i % 2u);
    of = i / 2u * kXcds + b % kXcds;
  } else {
    const uint32_t i = b - 2u * dealt, rest = main_blocks - dealt;
    r.half = i < rest ? 0 : 1;
    of = dealt + i - (uint32_t)r.half * rest;
  }
  const LineBlock lb = line_block(wm, n_main, 0, deal, cols, by_column, of);
  r.tile = lb.tile;
  r.col = lb.col;
  return r;
}

struct BatchBlock {
  int32_t leaf;  // its place in the table
  int32_t tile;  // feature tile
  int32_t half;  // of the tile, where main tiles are built in halves
  int32_t wg;    // workgroup of (leaf, tile)
};

// The leaf that owns workgroup column `col`: the last one that starts at or before it (a
// leaf without rows has no columns and is never the last such leaf of a live column).
GBDT_HD int32_t batch_leaf_of(const BatchLeaf* leaf, int32_t n_leaves, uint32_t col) {
  int32_t lo = 0, hi = n_leaves - 1;
  while (lo < hi) {
    const int32_t mid = (lo + hi + 1) >> 1;
    if (leaf[mid].first_wg <= col) {
      lo = mid;
    } else {
      hi = mid - 1;
    }
  }
  return lo;
}

GBDT_HD BatchBlock batch_block(const BatchLeaf* leaf, int32_t n_leaves, int32_t wm, int32_t n_main, int32_t wr,
                               int32_t deal, uint32_t cols, uint32_t b) {
  const LineBlock lb = line_block(wm, n_main, wr, deal, cols, true, b);
  BatchBlock r;
  r.leaf = batch_leaf_of(leaf, n_leaves, lb.col);
  r.tile = lb.tile;
  r.half = 0;
  r.wg = (int32_t)(lb.col - leaf[r.leaf].first_wg);
  return r;
}
GBDT_HD BatchBlock batch_half_block(const BatchLeaf* leaf, int32_t n_leaves, int32_t wm, int32_t n_main,
                                    int32_t deal, uint32_t cols, uint32_t b) {
  const HalfBlock hb = half_block(wm, n_main, deal, cols, true, b);
  BatchBlock r;
  r.leaf = batch_leaf_of(leaf, n_leaves, hb.col);
  r.tile = hb.tile;
  r.half = hb.half;
  r.wg = (int32_t)(hb.col - leaf[r.leaf].first_wg);
  return r;
}

#endif  // GBDT_BATCH_PLAN_H_
