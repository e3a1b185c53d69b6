// The reduction pass over the workgroups' partial histograms (Sec. 4, "final reduction
// program") and the sibling histogram by subtraction.  Included by gbdt_hist.hip only, after
// hist_build_kernels.h.
#ifndef GBDT_HIST_REDUCE_KERNELS_H_
#define GBDT_HIST_REDUCE_KERNELS_H_

#include <hip/hip_runtime.h>

#include <stdint.h>
#include <string.h>

#include "../../include/gbdt_hist.h"
#include "tile_plan.h"
#include "batch_plan.h"

namespace {

// ------------------------------------------------------------------ merge kernel

struct MergeArgs {
  const uint32_t* partials;
  gbdt_bin_t* out;
  TilePlan plan;
  int32_t n_features;
  int32_t n_bins;
  int32_t chunks_main;
  int32_t chunks_rem;
  int32_t halves;      // main tiles were built in halves (plan_halves)
  uint32_t* counters;  // the tiles' unit counters, set back to zero here; NULL: not used by the build
};

// Threads that share the partial blocks (chunks) of a cell, PARTS: 1, 2 or 4 where a cell has few chunks, 8 otherwise, and 32
// where there are few cells and many chunks (one or two tiles built by hundreds of workgroups: 8 would leave most of the machine
// idle).  A thread takes 4 neighbouring slots of a bin, with 16-byte loads, and has four chunks in flight, so with fewer than
// 4 * PARTS of them threads would wait for nothing.
constexpr int kMergePartsMost = 8, kMergePartsWide = 32;
template <int PARTS>
struct MergeShape {
  static constexpr int kQuads = PARTS < 8 ? 256 / PARTS : 16;  // groups of 4 slots of a workgroup
  static constexpr int kThreads = kQuads * PARTS;
  static constexpr int kCells = 4 * kQuads;
  // whole bins of a tile, of which every feature's run is then written together (12 bytes at a time is what
  // the others write)
  static constexpr bool kStaged = PARTS < 8;
};

// The "final reduction program" of Sec. 4: sums the partial histograms of the
// workgroups that shared a feature tile.  A workgroup takes kCells consecutive (bin,
// slot) pairs of one tile (slot fastest, so reads of a partial block are coalesced
// in runs of 32); PARTS threads per 4 pairs each sum every PARTS-th chunk in fp64, in chunk
// order, and the sub-sums are added in a fixed order: the result does not depend
// on scheduling.  Counts are summed as integers.  grid.y = tile.  (PARTS is a function of the launch's shape only.)
// Bound by the latency of its loads: four chunks are requested together.  (64 leaves of 1,500,000 x 500 x 255, 20 of them
// in 2 to 4 chunks: 57 us with 8 threads a cell and 12-byte stores, 25.5 with one and whole runs.)
template <int PARTS>
__device__ __forceinline__ void merge_cells(const MergeArgs& a) {
  using M = MergeShape<PARTS>;
  if (a.counters && blockIdx.x == 0 && threadIdx.x == 0) {
    const int32_t y = (int32_t)blockIdx.y;
    if (!a.halves) {
      a.counters[plan_counter_slot(y)] = 0u;
    } else {
      a.counters[plan_counter_slot(2 * y)] = 0u;  // (2 * n_main: the remainder tile's)
      if (y < a.plan.n_main) a.counters[plan_counter_slot(2 * y + 1)] = 0u;
    }
  }
  constexpr int kSums = PARTS > 1 ? M::kCells : 1;
  __shared__ double s_g[PARTS][kSums];
  __shared__ double s_h[PARTS][kSums];
  __shared__ uint32_t s_n[PARTS][kSums];
  __shared__ uint32_t s_run[M::kStaged ? 3 * M::kCells + 128 : 1];  // [slot][bin of the workgroup's][3], a word between slots
  const int32_t t = blockIdx.y;
  const int32_t w = plan_tile_width(a.plan, t);
  const int32_t slots = plan_slots(a.plan, w);
  const bool halved = a.halves && t < a.plan.n_main;
  const int32_t wb = halved ? 16 : w;  // width of the tile that a partial block is of
  const size_t hw = (size_t)plan_cells(a.plan, wb);
  const size_t main_block = (size_t)3 * plan_cells(a.plan, a.plan.wm);
  const uint32_t* p;
  int32_t chunks;
  if (t < a.plan.n_main) {
    p = a.partials + (size_t)t * a.chunks_main * main_block;
    chunks = a.chunks_main;
  } else {
    p = a.partials + (size_t)a.plan.n_main * a.chunks_main * main_block;
    chunks = a.chunks_rem;
  }
  const int quad = threadIdx.x % M::kQuads;
  const int part = threadIdx.x / M::kQuads;
  const int32_t e_first = blockIdx.x * M::kCells, e_end = a.n_bins * slots;
  if (e_first >= e_end) return;  // (the same for the whole workgroup: a narrow tile has fewer cells)
  const int32_t run_bins = M::kCells / slots;  // (staged: a multiple of the slots)
  const int32_t e0 = e_first + 4 * quad;
  // (a bin has a multiple of 16 slots, so the four cells are one bin's, and all live or none)
  const int32_t bin0 = e0 / slots, slot0 = e0 - bin0 * slots;
  double g[4] = {0.0, 0.0, 0.0, 0.0}, h[4] = {0.0, 0.0, 0.0, 0.0};
  uint32_t n[4] = {0u, 0u, 0u, 0u};
  if (e0 < e_end) {
    if (halved) p += (size_t)(slot0 >> 4) * chunks * 3 * hw;  // (all blocks of the first half, then those of the second)
    p += (size_t)plan_cell(a.plan, wb, bin0, halved ? slot0 & 15 : slot0) + (size_t)part * 3 * hw;
    const size_t step = (size_t)PARTS * 3 * hw;
    constexpr int kFlight = 4;
    for (int32_t c = part; c < chunks; c += kFlight * PARTS) {
      uint4 vg[kFlight], vh[kFlight], vn[kFlight];
#pragma unroll
      for (int i = 0; i < kFlight; ++i) {
        const size_t at = c + i * PARTS < chunks ? i * step : 0;  // (past the end: the first one again)
        vg[i] = *reinterpret_cast<const uint4*>(p + at);
        vh[i] = *reinterpret_cast<const uint4*>(p + at + hw);
        vn[i] = *reinterpret_cast<const uint4*>(p + at + 2 * hw);
      }
#pragma unroll
      for (int i = 0; i < kFlight; ++i) {
        if (c + i * PARTS < chunks) {
          g[0] += (double)__uint_as_float(vg[i].x);
          g[1] += (double)__uint_as_float(vg[i].y);
          g[2] += (double)__uint_as_float(vg[i].z);
          g[3] += (double)__uint_as_float(vg[i].w);
          h[0] += (double)__uint_as_float(vh[i].x);
          h[1] += (double)__uint_as_float(vh[i].y);
          h[2] += (double)__uint_as_float(vh[i].z);
          h[3] += (double)__uint_as_float(vh[i].w);
          n[0] += vn[i].x;
          n[1] += vn[i].y;
          n[2] += vn[i].z;
          n[3] += vn[i].w;
        }
      }
      p += kFlight * step;
    }
    if constexpr (PARTS > 1) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        s_g[part][4 * quad + k] = g[k];
        s_h[part][4 * quad + k] = h[k];
        s_n[part][4 * quad + k] = n[k];
      }
    }
  }
  auto stage = [&](int32_t bin, int32_t slot, double sg, double sh, uint32_t sn) {
    uint32_t* to = s_run + slot * (3 * run_bins + 1) + 3 * (bin - e_first / slots);
    to[0] = __float_as_uint((float)sg);
    to[1] = __float_as_uint((float)sh);
    to[2] = sn;
  };
  if constexpr (PARTS == 1) {
    if (e0 < e_end) {
#pragma unroll
      for (int k = 0; k < 4; ++k) stage(bin0, slot0 + k, g[k], h[k], n[k]);
    }
  } else {
    __syncthreads();
#pragma unroll 1
    for (int cell = threadIdx.x; cell < M::kCells; cell += M::kThreads) {
      const int32_t e = e_first + cell;
      if (e >= e_end) break;
      double sg = 0.0, sh = 0.0;
      uint32_t sn = 0;
#pragma unroll 8
      for (int q = 0; q < PARTS; ++q) {
        sg += s_g[q][cell];
        sh += s_h[q][cell];
        sn += s_n[q][cell];
      }
      const int32_t bin = e / slots, slot = e - bin * slots;
      if constexpr (M::kStaged) {
        stage(bin, slot, sg, sh, sn);
      } else {
        const int32_t f = plan_feature_of(a.plan, t, slot);
        if (f < a.n_features) {  // else: padding slot
          gbdt_bin_t r;
          r.grad = (float)sg;
          r.hess = (float)sh;
          r.count = sn;
          a.out[(size_t)f * a.n_bins + bin] = r;
        }
      }
    }
  }
  if constexpr (M::kStaged) {
    __syncthreads();
    const int32_t b0 = e_first / slots;
    const int32_t live = 3 * (a.n_bins - b0 < run_bins ? a.n_bins - b0 : run_bins);  // words of a feature's run
    const int32_t per = M::kThreads / slots;  // threads of a run (a slot count is at most 128)
    const int32_t slot = threadIdx.x / per, first = threadIdx.x % per;
    const int32_t f = plan_feature_of(a.plan, t, slot);
    if (f < a.n_features) {  // else: padding slot
      uint32_t* to = reinterpret_cast<uint32_t*>(a.out + (size_t)f * a.n_bins + b0);
      const uint32_t* from = s_run + slot * (3 * run_bins + 1);
      for (int32_t i = first; i < live; i += per) to[i] = from[i];
    }
  }
}

template <int PARTS>
__global__ void __launch_bounds__(MergeShape<PARTS>::kThreads) hist_merge_kernel(MergeArgs a) {
  merge_cells<PARTS>(a);
}

// Cells of a workgroup with `parts` threads a cell, and its threads.
inline int merge_wg_cells(int parts) { return parts < 8 ? 1024 / parts : 64; }
inline int merge_wg_threads(int parts) { return parts < 8 ? 256 : 16 * parts; }
// Cells of the widest tile: a matrix of few features has only a narrow one.  (Taken to be as wide as a main tile, 64 leaves of
// 700,000 x 5 x 64 with wide sums, 4 threads a cell and three of four workgroups without any: 8.6 us, 5.2 with 8.)
inline int64_t merge_tile_cells(const TilePlan& p, int32_t n_bins) {
  return (int64_t)n_bins * plan_slots(p, p.n_main ? p.wm : p.wr);
}
// Threads per cell for a reduction over n_tiles tiles (of all leaves) of `cells` cells at most, up to `chunks` partial blocks each.
inline int merge_parts(int64_t cells, int64_t n_tiles, int32_t chunks) {
  auto blocks = [&](int parts) { return (cells + merge_wg_cells(parts) - 1) / merge_wg_cells(parts) * n_tiles; };
  int parts = 1;
  while (parts < kMergePartsMost && (chunks > 4 * parts || blocks(parts) < 512)) parts *= 2;
  if (parts == kMergePartsMost && blocks(parts) < 512 && chunks >= 64) parts = kMergePartsWide;
  return parts;
}

// The same reduction for a batched launch: grid.z = leaf of the launch; its partial
// blocks start first_wg workgroup columns into the buffer, its histogram is the leaf's
// [n_features][n_bins] slice of the output.  A leaf without rows has no partial blocks
// and gets zeros; a leaf with a single workgroup per tile is skipped.
struct BatchMergeArgs {
  MergeArgs m;            // partials / out of leaf 0 of the launch; chunk counts unused
  uint64_t column_words;  // words of one workgroup column
  int32_t blocks_per_wg;  // partial blocks a workgroup wrote: 1, or 2 with wide accumulation
  BatchLeaf leaf[kBatchLeaves];
};

template <int PARTS>
__global__ void __launch_bounds__(MergeShape<PARTS>::kThreads) hist_merge_batch_kernel(BatchMergeArgs a) {
  const BatchLeaf lf = a.leaf[blockIdx.z];
  if (batch_wgs(lf) == 1u) return;  // written by the build kernel itself
  MergeArgs m = a.m;
  m.partials += (size_t)lf.first_wg * a.column_words;
  m.out += (size_t)batch_leaf_no(lf) * m.n_features * m.n_bins;
  m.chunks_main = (int32_t)batch_wgs(lf) * a.blocks_per_wg;
  m.chunks_rem = m.plan.wr ? m.chunks_main : 0;
  merge_cells<PARTS>(m);
}

// ----------------------------------------------------------------- unfuse kernel

// Marginals of the fused columns' joint histograms (see FusedCol): bin b of feature f is the sum
// of the joint bins v of its column with (v / stride) mod levels == b, v ascending, in fp64;
// bins that do not occur are zero.  One thread per (feature, bin).
__global__ void __launch_bounds__(256)
hist_unfuse_kernel(const gbdt_bin_t* __restrict__ joint, const FusedFeat* __restrict__ feats,
                   int32_t n_features, int32_t n_bins, gbdt_bin_t* __restrict__ out) {
  const int32_t e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n_features * n_bins) return;
  const int32_t f = e / n_bins;
  const int32_t b = e - f * n_bins;
  const FusedFeat ff = feats[f];
  gbdt_bin_t r;
  r.grad = 0.0f;
  r.hess = 0.0f;
  r.count = 0u;
  if (b < (int32_t)ff.levels) {
    const gbdt_bin_t* col = joint + (size_t)ff.col * kFusedCap;
    const int32_t stride = ff.stride, period = stride * (int32_t)ff.levels;
    double g = 0.0, h = 0.0;
    uint32_t n = 0;
    // the joint bins v = hi * period + b * stride + lo (lo < stride) in ascending order, sixteen at a
    // time: their loads are issued together (they do not depend on one another), then summed in order
    int32_t base = b * stride, lo = 0;
    while (base < kFusedCap) {
      gbdt_bin_t c[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int32_t v = base + lo;
        const bool ok = base < kFusedCap && v < kFusedCap;
        c[i].grad = 0.0f;
        c[i].hess = 0.0f;
        c[i].count = 0u;
        if (ok) c[i] = col[v];
        if (++lo == stride) {
          lo = 0;
          base += period;
        }
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        g += (double)c[i].grad;
        h += (double)c[i].hess;
        n += c[i].count;
      }
    }
    r.grad = (float)g;
    r.hess = (float)h;
    r.count = n;
  }
  out[e] = r;
}

// --------------------------------------------------------------- subtract kernel

// sibling = parent - child, element by element over [n_features][n_bins].
__global__ void __launch_bounds__(256)
hist_subtract_kernel(const gbdt_bin_t* parent, const gbdt_bin_t* child, gbdt_bin_t* sibling,
                     int32_t n) {
  const int32_t e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const gbdt_bin_t p = parent[e];
  const gbdt_bin_t c = child[e];
  gbdt_bin_t s;
  s.grad = p.grad - c.grad;
  s.hess = p.hess - c.hess;
  s.count = p.count - c.count;
  sibling[e] = s;
}

// Siblings of a tree level: large[j] = parent[parent_slot[j]] - small[j], histograms of n
// (bin, feature) elements; grid.y = j.  The slots travel as kernel arguments.
constexpr int kSiblingTable = 960;
struct SiblingTable {
  int32_t parent_slot[kSiblingTable];
};

__global__ void __launch_bounds__(256)
hist_siblings_kernel(const gbdt_bin_t* __restrict__ parents, const gbdt_bin_t* __restrict__ small,
                     gbdt_bin_t* __restrict__ large, int32_t n, SiblingTable t) {
  const int32_t e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const size_t j = blockIdx.y;
  const gbdt_bin_t p = parents[(size_t)t.parent_slot[j] * n + e];
  const gbdt_bin_t c = small[j * n + e];
  gbdt_bin_t s;
  s.grad = p.grad - c.grad;
  s.hess = p.hess - c.hess;
  s.count = p.count - c.count;
  large[j * n + e] = s;
}

// Histogram of an empty leaf: all zero.  (A fill kernel, not a memset node, so the
// call can be captured into a graph.)
__global__ void __launch_bounds__(256) hist_zero_kernel(gbdt_bin_t* hist, int32_t n) {
  const int32_t e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  gbdt_bin_t z;
  z.grad = 0.0f;
  z.hess = 0.0f;
  z.count = 0;
  hist[e] = z;
}

}  // namespace

#endif  // GBDT_HIST_REDUCE_KERNELS_H_
