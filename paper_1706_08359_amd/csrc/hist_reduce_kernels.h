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

constexpr int kMergeCells = 64;      // histogram cells per workgroup
constexpr int kMergeParts = 8;       // threads that share the chunks of a cell ...
constexpr int kMergePartsWide = 32;  // ... and when there are few cells and many chunks (one or two tiles built
                                     // by hundreds of workgroups): 8 would leave most of the machine idle
constexpr int kMergeQuads = kMergeCells / 4;  // a thread takes 4 neighbouring slots of a bin: 16-byte loads

// The "final reduction program" of Sec. 4: sums the partial histograms of the
// workgroups that shared a feature tile.  A workgroup takes 64 consecutive (bin,
// slot) pairs of one tile (slot fastest, so reads of a partial block are coalesced
// in runs of 32); PARTS threads per 4 pairs each sum every PARTS-th chunk in fp64, in chunk
// order, and the sub-sums are added in a fixed order: the result does not depend
// on scheduling.  Counts are summed as integers.  grid.y = tile.  (PARTS = 8 or 32;
// which one is a function of the launch's shape only.)  Bound by the latency of its loads: four chunks are
// requested together.
template <int PARTS>
__device__ __forceinline__ void merge_cells(const MergeArgs& a) {
  if (a.counters && blockIdx.x == 0 && threadIdx.x == 0) {
    const int32_t y = (int32_t)blockIdx.y;
    if (!a.halves) {
      a.counters[plan_counter_slot(y)] = 0u;
    } else {
      a.counters[plan_counter_slot(2 * y)] = 0u;  // (2 * n_main: the remainder tile's)
      if (y < a.plan.n_main) a.counters[plan_counter_slot(2 * y + 1)] = 0u;
    }
  }
  __shared__ double s_g[PARTS][kMergeCells];
  __shared__ double s_h[PARTS][kMergeCells];
  __shared__ uint32_t s_n[PARTS][kMergeCells];
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
  const int quad = threadIdx.x % kMergeQuads;
  const int part = threadIdx.x / kMergeQuads;
  const int32_t e0 = blockIdx.x * kMergeCells + 4 * quad;
  // (a bin has a multiple of 16 slots, so the four cells are one bin's, and all live or none)
  if (e0 < a.n_bins * slots) {
    const int32_t bin = e0 / slots;
    const int32_t slot = e0 - bin * slots;
    if (halved) p += (size_t)(slot >> 4) * chunks * 3 * hw;  // (all blocks of the first half, then those of the second)
    p += (size_t)plan_cell(a.plan, wb, bin, halved ? slot & 15 : slot) + (size_t)part * 3 * hw;
    double g[4] = {0.0, 0.0, 0.0, 0.0}, h[4] = {0.0, 0.0, 0.0, 0.0};
    uint32_t n[4] = {0u, 0u, 0u, 0u};
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
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      s_g[part][4 * quad + k] = g[k];
      s_h[part][4 * quad + k] = h[k];
      s_n[part][4 * quad + k] = n[k];
    }
  }
  __syncthreads();
  const int cell = threadIdx.x;
  const int32_t e = blockIdx.x * kMergeCells + cell;
  if (cell < kMergeCells && e < a.n_bins * slots) {
    const int32_t bin = e / slots;
    const int32_t f = plan_feature_of(a.plan, t, e - bin * slots);
    if (f < a.n_features) {  // else: padding slot
      double g = 0.0, h = 0.0;
      uint32_t n = 0;
#pragma unroll
      for (int q = 0; q < PARTS; ++q) {
        g += s_g[q][cell];
        h += s_h[q][cell];
        n += s_n[q][cell];
      }
      gbdt_bin_t r;
      r.grad = (float)g;
      r.hess = (float)h;
      r.count = n;
      a.out[(size_t)f * a.n_bins + bin] = r;
    }
  }
}

template <int PARTS>
__global__ void __launch_bounds__(kMergeQuads * PARTS) hist_merge_kernel(MergeArgs a) {
  merge_cells<PARTS>(a);
}

// Threads per cell for a reduction over `blocks` workgroups of 8 of them and up to
// `chunks` partial blocks per cell.
inline int merge_parts(int64_t blocks, int32_t chunks) {
  return (blocks < 512 && chunks >= 64) ? kMergePartsWide : kMergeParts;
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
__global__ void __launch_bounds__(kMergeQuads * PARTS) hist_merge_batch_kernel(BatchMergeArgs a) {
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
