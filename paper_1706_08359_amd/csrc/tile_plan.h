// Device layout of the binned feature matrix and of the local-memory histograms.
//
// The paper (Sec. 4, "Data Structure") bundles 4 one-byte features of a sample
// into one 4-byte word so that a thread never fetches a single byte, and stores
// those words tuple-major.  Here the bundle is kept (a lane loads 4, 8 or 16 bytes
// = that many features, twice as many with 4-bit bins, App. C.4) but words are laid
// out row-major inside FEATURE TILES of W bytes: tile t holds, for every row, W
// consecutive bytes.  A gathered leaf row then costs one contiguous W-byte
// segment per tile instead of one 4-byte word per cache line.
//
//   packed = [tile 0: n_rows x W_0 bytes][tile 1: n_rows x W_1 bytes] ...
//
// (from 4,096 rows on two tiles share such a region, row by row: "Lines" below).
// All tiles have the "main" width WM except possibly the last one, which is 16
// or 32 bytes wide when few feature bytes remain (so that padding stays small).
//
// Behind the tiles, and a slack the build kernels may read (and ignore) past the last
// tile, the matrix is stored ONCE MORE, column by column, one byte per value:
//
//   packed = [tiles][slack][column 0: stride bytes][column 1] ...     stride = n_rows rounded up to 256
//
// The row partition after a split looks at ONE feature of every row of a leaf; from the
// tiles that costs a whole 32- or 64-byte tile row per row, from a column one byte.  The
// copy doubles the resident matrix (triples it with 4-bit bins) -- memory this part has.
//
// Inside a tile, a lane loads VEC consecutive bytes of a row (W / 4 with 8-bit bins;
// 4 or 8 with 4-bit bins), so a row is LPR = W / VEC = 4 or 8 lane-chunks.  Byte i of the tile row
// is byte bl = i % VEC of lane-chunk j = i / VEC.  The lane splits its bytes
// into "byte-words" of 4 bin values each: with 8-bit bins byte-word bw is the
// loaded word bl / 4; with 4-bit bins each loaded word gives two byte-words, its
// low nibbles (features 2i) and its high nibbles (features 2i + 1): bw = 2 *
// (bl / 4) + half.  q = bl % 4 is the value's byte inside its byte-word.
//
// Histogram slot of a feature of the tile:  s = j + LPR * q + 4 * LPR * bw.
// The local-memory histogram and each partial block in the workspace are cells
// [page = s / 32][bin][s % 32]; one page row (32 cells of 8 bytes) spans all 32
// banks twice.  With this slot order the lanes the LDS serves together,
// which at any step work on pairwise different (j, q), fall into different
// banks whatever the bin values are (see build_tile).  A tile of 16 slots with 256 bins has rows of 16 cells
// (they span the banks once): half the cells to clear, drain and sum.
#ifndef GBDT_TILE_PLAN_H_
#define GBDT_TILE_PLAN_H_

#include <stdint.h>

#if defined(__HIPCC__)
#define GBDT_HD __host__ __device__ __forceinline__
#else
#define GBDT_HD inline
#endif

struct TilePlan {
  int32_t cap;        // bin capacity of the kernel variant: 16, 64 or 256
  int32_t nib;        // 1: 4-bit bins, two per byte
  int32_t wm;         // main tile width in bytes (64, or 32 when cap == 256)
  int32_t n_main;     // number of main tiles
  int32_t wr;         // width of the remainder tile in bytes (16 / 32), 0 if none
  int32_t row_bytes;  // n_main * wm + wr: packed bytes per row
  int32_t feat_bytes; // bytes of real feature data per row (before padding)
};

GBDT_HD TilePlan make_tile_plan(int32_t n_features, int32_t n_bins) {
  TilePlan p;
  p.nib = n_bins <= 16 ? 1 : 0;
  p.cap = n_bins <= 16 ? 16 : (n_bins <= 64 ? 64 : 256);
  p.wm = p.cap == 256 ? 32 : 64;
  p.feat_bytes = p.nib ? (n_features + 1) / 2 : n_features;
  p.n_main = p.feat_bytes / p.wm;
  int32_t rem = p.feat_bytes - p.n_main * p.wm;
  p.wr = 0;
  if (rem > p.wm / 2) {
    p.n_main += 1;  // more than half a tile left: pad it to a full tile
  } else if (rem > 0) {
    p.wr = rem <= 16 ? 16 : 32;
  }
  p.row_bytes = p.n_main * p.wm + p.wr;
  return p;
}

// Bytes behind the last tile that the build kernel may read (and ignore): its last epoch
// of a root leaf fetches whole row groups, up to one epoch (512 rows) of the widest tile
// past the end.
constexpr int64_t kPlanSlackBytes = 512 * 64;
GBDT_HD int64_t plan_column_stride(int64_t n_rows) { return (n_rows + 255) / 256 * 256; }
GBDT_HD int64_t plan_columns_base(const TilePlan& p, int64_t n_rows) {
  return (n_rows * (int64_t)p.row_bytes + kPlanSlackBytes + 255) / 256 * 256;
}
GBDT_HD int64_t plan_packed_bytes(const TilePlan& p, int64_t n_rows, int32_t n_features) {
  return plan_columns_base(p, n_rows) + (int64_t)n_features * plan_column_stride(n_rows);
}

// Lines.  Memory is fetched in lines of 128 bytes, and a tile row has 64 or 32: a leaf that is a
// small part of the matrix fetches two or four times the bytes it uses when every tile has a region
// of its own.  (Measured with a plain gather of listed rows: 5.8 TB/s of whole lines at any density, whether
// 32, 64 or 128 bytes of them are used.)  So two neighbouring main tiles share a region, one after
// the other inside a row of 128 or 64 bytes, and the build kernels run the workgroups that need the
// same line on the same XCD at the same time (batch_plan.h): one of them fetches it, the others find it in
// that XCD's L2.
// Build kernel, a region per tile -> shared: 8,000,000 x 500 x 64 bins, 50 / 25 / 12.5 % of the rows 657 / 368 / 202
// -> 467 / 243 / 136 us; 2,000,000 x 500 x 255 bins, 25 / 5 % 147 / 43 -> 122 / 32 us; 400,000 x 2,000 x 63
// bins, half of the rows 123 -> 101 us, all rows 176 -> 179 us.  (Four 32-byte tiles a line were
// better still for sparse leaves, 107 / 32 us, but the root then fetches its lines up to four times:
// 362 -> 413 us.)
// What is left over, a main tile without a partner and the remainder tile, shares a region only with 32-byte tiles:
// rows of 48 bytes (1,000,000 x 40 x 255: 32 leaves of a call 57 -> 46 us, the root 38 either way).  With
// 64-byte tiles the rows would have 80 or 96 bytes and two or three of eight would lie across two lines:
// 1,000,000 x 150 x 16 bins, root 47 us with a region each and 62 with one, 32 leaves 53 and 52;
// 300,000 x 70 x 64, root 24.1 and 26.4, 32 leaves 29.7 and 30.1.
// Small matrices keep one region per tile: they fit the caches anyway, and the build may
// read up to kEpochRows - 1 rows past the last one, which have to lie inside the buffer: with 128-byte
// rows that is more than the slack, but with kPlanLinesMinRows rows and the features of two
// tiles the columns behind it are longer still.  So do the largest, whose byte offsets in a
// region of 128-byte rows would not fit 32 bits.
constexpr int64_t kPlanLinesMinRows = 4096;
constexpr int64_t kPlanLinesMaxRows = ((int64_t)1 << 25) - 1024;
GBDT_HD int32_t plan_line_tiles(int64_t n_rows) {  // main tiles per row of a region: 1 or 2
  return n_rows >= kPlanLinesMinRows && n_rows <= kPlanLinesMaxRows ? 2 : 1;
}
// ... and whether a main tile left over alone shares its region with the remainder tile.
GBDT_HD bool plan_leftover_shared(int32_t wm, int32_t n_main, int32_t wr) {
  return (n_main & 1) != 0 && wr != 0 && wm == 32;
}
struct TileAt {
  int64_t off;     // byte offset of the tile's first row
  int32_t stride;  // bytes from a row to the next
  bool shared;     // the region holds another tile too
};
GBDT_HD TileAt plan_tile_at(int32_t wm, int32_t n_main, int32_t wr, int64_t n_rows, int32_t line_tiles, int32_t t) {
  TileAt a;
  const int32_t paired = n_main & ~1;  // main tiles that share a region with another main tile
  int32_t first = t;                   // the region's first tile; the tiles in front of it are main tiles
  a.stride = t < n_main ? wm : wr;
  if (line_tiles > 1 && t < paired) {
    first = t & ~1;
    a.stride = 2 * wm;
  } else if (line_tiles > 1 && plan_leftover_shared(wm, n_main, wr)) {
    first = paired;
    a.stride = wm + wr;
  }
  a.off = n_rows * ((int64_t)first * wm) + (int64_t)(t - first) * wm;
  a.shared = a.stride > (t < n_main ? wm : wr);
  return a;
}

GBDT_HD int32_t plan_n_tiles(const TilePlan& p) { return p.n_main + (p.wr ? 1 : 0); }
// what workgroups of a build take one each of: tiles, or their halves
GBDT_HD int32_t plan_n_parts(const TilePlan& p, bool halves) { return (halves ? 2 * p.n_main : p.n_main) + (p.wr ? 1 : 0); }
GBDT_HD int32_t plan_tile_width(const TilePlan& p, int32_t t) { return t < p.n_main ? p.wm : p.wr; }
// features (= slots) held by a tile of width w
GBDT_HD int32_t plan_slots(const TilePlan& p, int32_t w) { return p.nib ? 2 * w : w; }
// bytes a lane loads from a row of a tile of width w: a quarter of the row with 8-bit
// bins; with 4-bit bins at most 8 (16 bin values)
GBDT_HD int32_t plan_vec(const TilePlan& p, int32_t w) { return p.nib ? (w == 16 ? 4 : 8) : w / 4; }
// pages of 32 slots in the histogram of a tile of width w
GBDT_HD int32_t plan_pages(const TilePlan& p, int32_t w) { return (plan_slots(p, w) + 31) / 32; }
// cells from a bin to the next in the histogram of a tile of width w
GBDT_HD constexpr int32_t plan_pitch(int32_t cap, int32_t slots) { return cap == 256 && slots == 16 ? 16 : 32; }
// cells ((bin, slot) pairs, padding included) of the histogram of a tile of width w
GBDT_HD int32_t plan_cells(const TilePlan& p, int32_t w) {
  return plan_pages(p, w) * p.cap * plan_pitch(p.cap, plan_slots(p, w));
}
// index of cell (bin, slot) inside a histogram / partial block of a tile of width w
GBDT_HD int32_t plan_cell(const TilePlan& p, int32_t w, int32_t bin, int32_t slot) {
  const int32_t pitch = plan_pitch(p.cap, plan_slots(p, w));
  return (slot >> 5) * p.cap * 32 + bin * pitch + (slot & 31);
}

// With wide accumulation a pair of cells is kept for every (bin, slot), and a 32-byte tile of 256 bins fills most of a
// CU's local memory: one workgroup a CU.  Its main tiles are then built in HALVES, by different workgroups, two a CU: half h
// takes the slots 16 h .. 16 h + 15, which are the byte-word h of every lane-chunk, and has the cells of a 16-byte tile.
// (2,270,000 x 137 x 255, root 302 us with whole tiles, 217 in halves, 10 % of the rows 54 and 45; 10,500,000 x 28 x 255,
// root 269 and 218, half of the rows 157 and 123.)  Not so sparse leaves of a matrix of one tile, which are bound by the
// lines they fetch, bins and statistics, now twice: a tenth of 10,500,000 x 28 x 255 49.7 us whole, 53.5 in halves; 32 leaves
// of 4,000,000 x 28 x 255, all its rows, in a call 217 and 225.  (One 16-byte tile has nothing to halve, but the kernel with two
// workgroups a CU has more rows in flight than its lines bear too: a tenth of 10,500,000 x 16 x 255 39.7 us with one,
// 48.5 with two, 2 % 24.1 and 29.1.)  Nor many sparse rows of one tile and a remainder: 32 leaves of 4,000,000 x 33 x 255, half
// of its rows, 133 us whole, 177 in halves, a tenth of them in one list 36.9 and 42.7; but few, 32 leaves of a tenth of
// 1,000,000 x 33 x 255, 31.1 and 23.2.
// A matrix of two or three tiles that is too big for the two halves' lines to meet in the caches (large: see rows_of_leaf): many
// sparse rows of one list stay whole, 5 % of 20,000,000 x 64 x 255 75.9 us, 94.4 in halves, x 70 97 and 124, a tenth of 10,000,000 x 96
// 92.7 and 112 (19 % of 20,000,000 x 70 278 and 264); of a batch with two full tiles only, 32 leaves of half of 20,000,000 x 64 592 and
// 741, x 70 1111 and 888 (64 leaves of all 2184 and 2331), 64 of all of 10,000,000 x 96 1108 and 1039.  With four tiles halves win.
// how the rows of a build lie in the matrix:
constexpr int kRowsDense = 0, kRowsSparse = 1, kRowsSparseMany = 2, kRowsLargeBatch = 3, kRowsLargeList = 4;
GBDT_HD bool plan_halves(const TilePlan& p, bool wide, int rows) {
  if (!wide || p.cap != 256) return false;
  const int n_tiles = p.n_main + (p.wr ? 1 : 0);
  if (n_tiles > 3) return true;
  if (n_tiles == 1) return rows < kRowsSparse;
  return rows < (n_tiles == 3 ? kRowsLargeList : (p.wr ? kRowsSparseMany : kRowsLargeBatch));
}

struct FeatureSlot {
  int32_t tile;
  int32_t slot;
};

// Where feature f lives: which tile, and which slot of that tile's histogram.
GBDT_HD FeatureSlot plan_locate(const TilePlan& p, int32_t f) {
  int32_t fb = p.nib ? (f >> 1) : f;  // byte of the row holding f
  int32_t t = fb / p.wm;
  if (t >= p.n_main) t = p.n_main;  // remainder tile
  int32_t w = plan_tile_width(p, t);
  int32_t i = fb - t * p.wm;  // byte inside the tile row
  int32_t vec = plan_vec(p, w);
  int32_t lpr = w / vec;
  int32_t j = i / vec;
  int32_t bl = i - j * vec;  // byte inside the lane-chunk
  int32_t bw = p.nib ? (2 * (bl >> 2) + (f & 1)) : (bl >> 2);
  int32_t q = bl & 3;
  FeatureSlot r;
  r.tile = t;
  r.slot = j + lpr * q + 4 * lpr * bw;
  return r;
}

// Inverse of plan_locate: the feature held by `slot` of tile t (may be >= n_features
// for padding slots).
GBDT_HD int32_t plan_feature_of(const TilePlan& p, int32_t t, int32_t slot) {
  int32_t w = plan_tile_width(p, t);
  int32_t vec = plan_vec(p, w);
  int32_t lpr = w / vec;
  int32_t bw = slot / (4 * lpr);
  int32_t rest = slot - bw * 4 * lpr;
  int32_t q = rest / lpr;
  int32_t j = rest - q * lpr;
  if (p.nib) {
    int32_t bl = 4 * (bw >> 1) + q;
    return 2 * (t * p.wm + j * vec + bl) + (bw & 1);
  }
  return t * p.wm + j * vec + 4 * bw + q;
}

// The unit counter of tile t in the head of a scratch buffer (65,536 words): neighbouring tiles'
// counters lie 256 bytes apart, so that the device-scope atomics of a launch's workgroups do not
// all queue at the memory channel of one cache line.
GBDT_HD int32_t plan_counter_slot(int32_t t) { return (t & 1023) * 64 + (t >> 10); }

#endif  // GBDT_TILE_PLAN_H_
