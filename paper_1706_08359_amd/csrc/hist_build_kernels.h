// Re-layout of the bin matrix and the histogram build kernels (single leaf and batched):
// Alg. 1 / Sec. 4 / App. A.1 of arXiv 1706.08359 for gfx950.  Included by gbdt_hist.hip only.
#ifndef GBDT_HIST_BUILD_KERNELS_H_
#define GBDT_HIST_BUILD_KERNELS_H_

#include <hip/hip_runtime.h>

#include <stdint.h>
#include <string.h>

#include <type_traits>
#include <utility>

#include "../../include/gbdt_hist.h"
#include "tile_plan.h"
#include "batch_plan.h"
#include "cell_format.h"

namespace {

// ------------------------------------------------------------------ pack kernel

// Both device layouts of the matrix from one reading of it: the feature tiles (tile_plan.h), and
// the column-major copy behind them.  A workgroup takes 128 rows x 128 features: a
// thread reads 16 consecutive features of a row (any alignment: rows are n_features bytes apart) and
// writes them to their tile as they are, 16 bytes at a time (8 with 4-bit bins); a copy goes through local
// memory, from where every thread takes 16 rows of 4 features, turns them with byte permutes
// and writes 16 rows of a column, eight threads a whole line of 128 bytes.  Bound by memory:
// 400,000 x 2,000 is 800 MB read and 1.6 GB written.  (Two kernels of 4-byte words put together from single
// bytes took 0.80 ms for the tiles and 1.03 ms for the columns; this one takes 0.52, 4.6 TB/s.)
// STREAM: what is written is marked as not needed soon.  Copies that the memory-side cache cannot hold are better not kept in
// any cache: they would only be written back while the root is built (400,000 x 2,000 x 63: 575 -> 522 us, and the root build
// right behind it 222 -> 192); smaller ones are found there by that build (4,000,000 x 28 x 255, 224 MB: 64 us, 67 with the
// mark).
// grid = (row blocks, feature blocks).
constexpr int kPackRows = 128, kPackFeatures = 128;
constexpr int kPackPitch = kPackFeatures / 4 + 1;  // 4-byte words from a row to the next in local memory

// 16 bytes of src from byte `at` on, as far as there are `valid` of them (the rest 0), each & mask4's byte.
// total: bytes src has.
__device__ __forceinline__ uint4 pack_load16(const uint8_t* __restrict__ src, int64_t at, int64_t total,
                                             int32_t valid, uint32_t mask4) {
  uint32_t w[4] = {0u, 0u, 0u, 0u};
  if (valid > 0) {
    if (at + 16 <= total) {
      __builtin_memcpy(w, src + at, 16);  // (may reach into the next row: masked below)
    } else {
      for (int i = 0; i < 16 && at + i < total; ++i) w[i >> 2] |= (uint32_t)src[at + i] << (8 * (i & 3));
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int32_t nb = valid - 4 * k;  // valid bytes of this word
    const uint32_t keep = nb >= 4 ? ~0u : (nb <= 0 ? 0u : (1u << (8 * nb)) - 1u);
    w[k] &= keep & mask4;
  }
  return make_uint4(w[0], w[1], w[2], w[3]);
}

template <bool STREAM, typename WORDS>
__device__ __forceinline__ void pack_store(uint8_t* to, const uint32_t (&v)[sizeof(WORDS) / 4]) {
  WORDS w;
  __builtin_memcpy(&w, v, sizeof w);
  if constexpr (STREAM) {
    __builtin_nontemporal_store(w, reinterpret_cast<WORDS*>(to));
  } else {
    *reinterpret_cast<WORDS*>(to) = w;
  }
}

template <bool NIB, bool STREAM>
__global__ void __launch_bounds__(256)
pack_kernel(const uint8_t* __restrict__ src, int64_t n_rows, int32_t n_features, TilePlan plan, int32_t line_tiles,
            uint32_t mask4, uint8_t* __restrict__ tiles, uint8_t* __restrict__ cols, int64_t col_stride) {
  __shared__ uint32_t t[kPackRows * kPackPitch];
  const int tid = threadIdx.x;
  const int64_t r0 = (int64_t)blockIdx.x * kPackRows;
  const int32_t f0 = (int32_t)blockIdx.y * kPackFeatures;
  const int64_t total = n_rows * n_features;
  typedef uint32_t Words2 __attribute__((ext_vector_type(2)));
  typedef uint32_t Words4 __attribute__((ext_vector_type(4)));
  constexpr int kSteps = kPackRows / 32;  // 8 threads a row, 32 rows a step
  const int j = tid & 7;
  const int32_t f = f0 + 16 * j;
  uint4 v[kSteps];
#pragma unroll
  for (int i = 0; i < kSteps; ++i) {
    const int64_t r = r0 + (tid >> 3) + 32 * i;
    v[i] = r < n_rows ? pack_load16(src, r * n_features + f, total, n_features - f, mask4)
                      : make_uint4(0u, 0u, 0u, 0u);
  }
  const int32_t fb = NIB ? f >> 1 : f;  // this thread's first byte of the (virtual, padded) packed row
  if (fb < plan.row_bytes) {
    int32_t tile = fb / plan.wm;
    if (tile > plan.n_main) tile = plan.n_main;
    const TileAt at = plan_tile_at(plan.wm, plan.n_main, plan.wr, n_rows, line_tiles, tile);
    uint8_t* dst = tiles + at.off + (fb - tile * plan.wm);
#pragma unroll
    for (int i = 0; i < kSteps; ++i) {
      const int64_t r = r0 + (tid >> 3) + 32 * i;
      if (r >= n_rows) break;
      if (NIB) {  // features 2i, 2i + 1 -> low and high half of byte i
        const uint32_t x0 = v[i].x | (v[i].x >> 4), x1 = v[i].y | (v[i].y >> 4);
        const uint32_t x2 = v[i].z | (v[i].z >> 4), x3 = v[i].w | (v[i].w >> 4);
        const uint32_t o[2] = {__builtin_amdgcn_perm(x1, x0, 0x06040200u), __builtin_amdgcn_perm(x3, x2, 0x06040200u)};
        pack_store<STREAM, Words2>(dst + r * at.stride, o);
      } else {
        const uint32_t o[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
        pack_store<STREAM, Words4>(dst + r * at.stride, o);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < kSteps; ++i) {
    uint32_t* row = t + ((tid >> 3) + 32 * i) * kPackPitch + 4 * j;
    row[0] = v[i].x;
    row[1] = v[i].y;
    row[2] = v[i].z;
    row[3] = v[i].w;
  }
  __syncthreads();
  // 16 rows (group rg) of the 4 features of word w
  const int rg = tid & 7, w = tid >> 3;
  const int32_t fw = f0 + 4 * w;
  if (fw >= n_features) return;
  uint32_t out[4][4];  // [feature][4 rows each]
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    uint32_t a[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = t[(16 * rg + 4 * q + i) * kPackPitch + w];
    const uint32_t lo01 = __builtin_amdgcn_perm(a[1], a[0], 0x05010400u);  // a0.0 a1.0 a0.1 a1.1
    const uint32_t hi01 = __builtin_amdgcn_perm(a[1], a[0], 0x07030602u);  // a0.2 a1.2 a0.3 a1.3
    const uint32_t lo23 = __builtin_amdgcn_perm(a[3], a[2], 0x05010400u);
    const uint32_t hi23 = __builtin_amdgcn_perm(a[3], a[2], 0x07030602u);
    out[0][q] = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u);
    out[1][q] = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u);
    out[2][q] = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u);
    out[3][q] = __builtin_amdgcn_perm(hi23, hi01, 0x07060302u);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k)  // (rows past n_rows fall into the column's padding: its stride is a multiple of 256)
    if (fw + k < n_features)
      pack_store<STREAM, Words4>(cols + (int64_t)(fw + k) * col_stride + r0 + 16 * rg, out[k]);
}

// ------------------------------------------------------------- fused columns
//
// Features with few distinct bins can share one histogram column: the bins b_1 .. b_m of m
// features with L_1 .. L_m levels (L_1 * ... * L_m <= 64) are stored as ONE byte
// v = b_1 + L_1 * (b_2 + L_2 * (...)), the build kernel accumulates the column's joint
// histogram over v with ONE local-memory atomic per row, and each feature's histogram is a
// marginal of it (hist_unfuse_kernel).  The paper stores features of at most 16 bins in 4 bits
// to halve the bytes (App. C.4) and spreads features that use few bins over MORE counters to
// cut atomic conflicts (Alg. 3, App. A.3); on this part conflicts cost nothing and the number
// of atomic instructions is what bounds the build, so few-level features are merged into FEWER
// counters instead.  A constant feature (one level) rides along for free.
constexpr int kFusedCap = 64;      // joint levels per column: the bin capacity of the kernel variant used
constexpr int kFusedMaxParts = 6;  // features per column: 2^6 = 64

struct FusedCol {  // one column of the fused layout
  int32_t feature[kFusedMaxParts];  // -1: unused
  uint8_t stride[kFusedMaxParts];   // L_1 * ... * L_(k-1)
  uint8_t n_parts;
  uint8_t pad;
};
struct FusedFeat {  // where a feature went
  int32_t col;
  uint8_t stride;
  uint8_t levels;  // bins 0 .. levels - 1 occur
  uint8_t pad[2];
};

// Largest bin value of every feature over the rows [0, n_rows) of a row-major matrix of total_rows rows (maxima
// start at zero).  A thread takes 16 consecutive features; 1 << lane_bits of them cover a row (up to 1024
// features; wider matrices take more blocks in y) and the others of the workgroup take other rows,
// 8 in flight each; maxima are kept per byte in pairs of 16-bit halves, combined in local memory, and only one that
// exceeds what is known already is sent out with an atomic.  grid = (row stripes, blocks of 1024 features).
constexpr int kMaxFeatures = 1024;
constexpr int kMaxFlight = 8;
__global__ void __launch_bounds__(256)
feature_max_kernel(const uint8_t* __restrict__ src, int64_t n_rows, int64_t total_rows, int32_t n_features,
                   int32_t lane_bits, uint32_t* __restrict__ max_out) {
  typedef unsigned short half2u __attribute__((ext_vector_type(2)));
  __shared__ uint32_t s_max[kMaxFeatures];
  const int32_t f_block = (int32_t)blockIdx.y * kMaxFeatures;
  const int32_t fl = 16 * (int32_t)(threadIdx.x & ((1u << lane_bits) - 1u));  // first feature, in the block
  const int32_t f = f_block + fl;
  const int32_t rows_per_block = 256 >> lane_bits;
  for (int i = threadIdx.x; i < kMaxFeatures; i += 256) s_max[i] = 0u;
  __syncthreads();
  if (f < n_features) {
    const int64_t total = total_rows * n_features;
    const int64_t stripe = (int64_t)gridDim.x * rows_per_block;
    uint32_t even[4] = {0u, 0u, 0u, 0u}, odd[4] = {0u, 0u, 0u, 0u};  // bytes 0, 2 and 1, 3 of every word
    auto larger = [](uint32_t x, uint32_t y) {
      half2u p, q;
      __builtin_memcpy(&p, &x, 4);
      __builtin_memcpy(&q, &y, 4);
      const half2u m = __builtin_elementwise_max(p, q);
      uint32_t r;
      __builtin_memcpy(&r, &m, 4);
      return r;
    };
    for (int64_t r = (int64_t)blockIdx.x * rows_per_block + (threadIdx.x >> lane_bits); r < n_rows;
         r += kMaxFlight * stripe) {
      uint4 v[kMaxFlight];
#pragma unroll
      for (int i = 0; i < kMaxFlight; ++i) {
        const int64_t ri = r + i * stripe < n_rows ? r + i * stripe : r;
        v[i] = pack_load16(src, ri * n_features + f, total, n_features - f, ~0u);
      }
#pragma unroll
      for (int i = 0; i < kMaxFlight; ++i) {
        const uint32_t w[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          even[k] = larger(even[k], w[k] & 0x00ff00ffu);
          odd[k] = larger(odd[k], (w[k] >> 8) & 0x00ff00ffu);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int k = i >> 2, b = i & 3;
      atomicMax(&s_max[fl + i], ((b & 1 ? odd[k] : even[k]) >> (b & 2 ? 16 : 0)) & 0xffffu);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kMaxFeatures && f_block + i < n_features; i += 256) {
    uint32_t* known = max_out + f_block + i;
    if (s_max[i] > __hip_atomic_load(known, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(known, s_max[i]);
  }
}

// Copies words, also to page-locked host memory.
__global__ void __launch_bounds__(256)
words_copy_kernel(const uint32_t* __restrict__ from, int32_t n, uint32_t* __restrict__ to) {
  const int32_t i = (int32_t)(blockIdx.x * 256 + threadIdx.x);
  if (i < n) to[i] = from[i];
}

// The fused layout: feature tiles with a region each (whatever the rows: none are shared), as pack_kernel writes
// those of a small matrix of n_cols one-byte features, a byte being the joint value of its column.  One thread per 4-byte word.
__global__ void __launch_bounds__(256)
pack_fused_kernel(const uint8_t* __restrict__ src, int64_t n_rows, int32_t n_features, TilePlan plan,
                  const FusedCol* __restrict__ cols, int32_t n_cols, uint8_t* __restrict__ dst) {
  const int32_t t = blockIdx.y;
  const int32_t w = plan_tile_width(plan, t);
  const int32_t lpr = w >> 2;
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n_rows * lpr) return;
  const int64_t r = q / lpr;
  const int32_t j = (int32_t)(q - r * lpr);
  const int64_t tile_off = n_rows * ((int64_t)t * plan.wm);
  const uint8_t* row = src + r * (int64_t)n_features;
  uint32_t word = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int32_t c = t * plan.wm + 4 * j + i;
    uint32_t v = 0;
    if (c < n_cols) {
      const FusedCol col = cols[c];
      for (int k = 0; k < col.n_parts; ++k) v += (uint32_t)row[col.feature[k]] * col.stride[k];
      v &= (uint32_t)(kFusedCap - 1);
    }
    word |= v << (8 * i);
  }
  *reinterpret_cast<uint32_t*>(dst + tile_off + r * w + 4 * j) = word;
}

// The same for matrices of up to kFuseStageFeatures features: a workgroup stages kFuseStageRows whole rows in
// local memory and gathers the parts of its columns from there, every thread one word of the packed row
// for 8 rows at a time, so that a column's description is read once for them.  (Gathered byte by byte
// from memory, 3,000,000 x 700 took 7.2 ms; staged 1.7.)
constexpr int kFuseStageRows = 16;
constexpr int kFuseStageFeatures = 4096;
__global__ void __launch_bounds__(256)
pack_fused_staged_kernel(const uint8_t* __restrict__ src, int64_t n_rows, int32_t n_features, TilePlan plan,
                         const FusedCol* __restrict__ cols, int32_t n_cols, uint8_t* __restrict__ dst) {
  extern __shared__ __align__(16) uint8_t rows[];  // [kFuseStageRows][n_features]
  const int64_t r0 = (int64_t)blockIdx.x * kFuseStageRows;
  const int32_t nr = n_rows - r0 < kFuseStageRows ? (int32_t)(n_rows - r0) : kFuseStageRows;
  const int32_t bytes = nr * n_features;
  const uint8_t* from = src + r0 * n_features;
  for (int32_t at = 16 * (int32_t)threadIdx.x; at < bytes; at += 16 * 256) {
    if (at + 16 <= bytes) {
      uint4 v;
      __builtin_memcpy(&v, from + at, 16);
      *reinterpret_cast<uint4*>(rows + at) = v;
    } else {
      for (int32_t i = at; i < bytes; ++i) rows[i] = from[i];
    }
  }
  __syncthreads();
  constexpr int kRows = 8;  // rows a thread takes at a time
  const int32_t n_words = plan.row_bytes >> 2;
  for (int32_t item = (int32_t)threadIdx.x; item < n_words * (kFuseStageRows / kRows); item += 256) {
    const int32_t part = item / n_words, wd = item - part * n_words;
    if (part * kRows >= nr) break;
    uint32_t word[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) word[r] = 0u;
    for (int i = 0; i < 4; ++i) {
      const int32_t c = 4 * wd + i;
      if (c >= n_cols) break;
      const FusedCol col = cols[c];
      uint32_t v[kRows];
#pragma unroll
      for (int r = 0; r < kRows; ++r) v[r] = 0u;
#pragma unroll
      for (int k = 0; k < kFusedMaxParts; ++k) {
        if (k < col.n_parts) {
          const int32_t f = col.feature[k] + part * kRows * n_features;
#pragma unroll
          for (int r = 0; r < kRows; ++r)  // (rows past the last one: any staged byte, never stored)
            v[r] += (uint32_t)rows[part * kRows + r < nr ? f + r * n_features : 0] * col.stride[k];
        }
      }
#pragma unroll
      for (int r = 0; r < kRows; ++r) word[r] |= (v[r] & (uint32_t)(kFusedCap - 1)) << (8 * i);
    }
    const TileAt at = plan_tile_at(plan.wm, plan.n_main, plan.wr, n_rows, 1, 4 * wd / plan.wm);
    uint8_t* out = dst + at.off + (4 * wd) % plan.wm + (r0 + part * kRows) * at.stride;
#pragma unroll
    for (int r = 0; r < kRows; ++r)
      if (part * kRows + r < nr) *reinterpret_cast<uint32_t*>(out + (int64_t)r * at.stride) = word[r];
  }
}

// ----------------------------------------------------------- histogram build kernel

struct BuildArgs {
  const uint8_t* packed;
  const int32_t* idx;  // NULL: rows 0..n_leaf-1
  const float* grad;
  const float* hess;
  int32_t stats_by_pos;  // grad / hess are indexed by leaf position (gathered beforehand), not by row id
  uint32_t* partials;  // one [3][cells] block of words per workgroup
  uint32_t* counters;  // per tile: the next unit of work to hand out
  int64_t n_rows;
  int64_t n_leaf;
  int32_t n_main;       // main tiles
  int32_t wr;           // remainder tile width, 0 if none
  int32_t line_tiles;   // main tiles that share a region of the matrix (tile_plan.h)
  int32_t deal;         // order of the launch's blocks (batch_plan.h)
  int32_t wgs;          // workgroups per tile
  int32_t chunks;       // partial blocks per tile: wgs, or 2 * wgs with wide accumulation
  int32_t first_epochs; // 0, or the length of every workgroup's first unit
  int32_t unit_epochs;  // consecutive epochs a workgroup takes at a time
  int32_t fixed_stride; // 0: units from the tile's counter; else unit u is followed by u + this
  gbdt_bin_t* direct_out;  // wgs == 1 only: the histogram itself, written by the build kernel
  int32_t n_features;
  int32_t n_bins;
};

constexpr int kUnitEpochs = 4;  // consecutive epochs a workgroup takes from its group's counter (>= 3)

__device__ __forceinline__ float pow2f(int k) { return __uint_as_float((uint32_t)(k + 127) << 23); }

// acc + scale * (the sum of a cell, above its count) for any sum, each half of the cell exactly converted; scale is that of the cell
// as a whole, 2^kCountBits more of it.
__device__ __forceinline__ double add_wide_sum(double acc, uint32_t lo, uint32_t hi, double scale) {
  acc = fma((double)(int32_t)hi, scale * 4294967296.0, acc);
  return fma((double)(lo & ~((1u << kCountBits) - 1u)), scale, acc);
}
// ... and back, exactly, for |i| < 2^51: an addition and a subtraction instead of two conversions, a scaling and an
// addition.
__device__ __forceinline__ double i64_to_f64(long long i) {
  return __longlong_as_double(i + 0x4338000000000000LL) - 6755399441055744.0;
}

// Sum over the lanes of a wavefront with DPP moves (no LDS traffic); the total
// arrives in lane 63.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_add(float v) {
  const int t = __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROW_MASK, 0xf, false);
  return v + __int_as_float(t);
}
__device__ __forceinline__ float sum_in_8(float v) {  // every lane: sum of its aligned group of 8
  v = dpp_add<0xb1, 0xf>(v);   // quad_perm [1,0,3,2]
  v = dpp_add<0x4e, 0xf>(v);   // quad_perm [2,3,0,1]
  v = dpp_add<0x141, 0xf>(v);  // row_half_mirror
  return v;
}
__device__ __forceinline__ float wave_sum_to_lane63(float v) {
  v = sum_in_8(v);
  v = dpp_add<0x140, 0xf>(v);  // row_mirror: every lane holds the sum of its row of 16
  v = dpp_add<0x142, 0xa>(v);  // row_bcast15: rows 1 and 3 add the row before
  v = dpp_add<0x143, 0xc>(v);  // row_bcast31: rows 2 and 3 add lane 31 (rows 0 + 1)
  return v;
}

// Where a workgroup that is the only one of its (leaf, tile) writes the finished
// histogram itself instead of a partial block for the reduction pass (hist == NULL:
// partial block).
struct DirectOut {
  gbdt_bin_t* hist;  // [n_features][n_bins] of the leaf
  int32_t tile, wm, n_main, wr;
  int32_t first_slot;  // of the tile, of the workgroup's histogram: 0, or 16 for a second half
  int32_t n_features, n_bins;
};

// Compile-time shape of the work of one wavefront on a tile of width W.
template <int CAP, int W, bool NIB, int NT>
struct TileShape {
  static constexpr int VEC = NIB ? (W == 16 ? 4 : 8) : W / 4;  // bytes a lane loads: 4, 8 or 16
  static constexpr int NWORD = VEC / 4;             // 32-bit words a lane loads
  static constexpr int LPR = W / VEC;               // lanes per row
  static constexpr int RPW = 64 / LPR;              // rows per wavefront load
  static constexpr int NBW = NWORD * (NIB ? 2 : 1); // byte-words (4 bin values each) per lane
  static constexpr int SLOTS = 4 * LPR * NBW;       // features of the tile
  static constexpr int PAGES = (SLOTS + 31) / 32;
  static constexpr int PITCH = plan_pitch(CAP, SLOTS);  // cells from a bin to the next
  static constexpr int CELLS = PAGES * CAP * PITCH;
  static constexpr int NW = NT / 64;
  static constexpr int PP = CELLS / NT;             // cells drained by one thread
  static constexpr int GPE = 64 / RPW;              // row groups per wavefront per epoch
  static_assert(NT == kEpochRows, "an epoch gives every lane one row of its own");
  static_assert(CELLS % NT == 0, "every thread drains the same number of cells");
  static_assert(LPR == 4 || LPR == 8, "a row is shared by a quad or by two quads");
};

// This workgroup's share of the histogram of leaf positions [0, end) for one feature
// tile, accumulated in its local memory and then written out as one partial block.
//
// Lane mapping.  A lane loads VEC bytes of a tile row, so a row is LPR = W / VEC
// lane-chunks and a wavefront load covers RPW = 64 / LPR rows: lane = rho * LPR + j
// loads chunk j of row rho.  The chunk's bin values are then handled in steps, 4 per
// byte-word, and the order of the 4 steps is rotated by the lane's row: in step k
// the lane takes byte q = (rho + k) mod 4.  This is the rotation of Alg. 2 (p = (l +
// s) mod 4 there) used for a stronger purpose: with slot = j + LPR * q (+ a
// compile-time term per byte-word) and cells laid out [page][bin][32 slots], the 16
// lanes whose 64-bit atomics the LDS serves together address 16 different,
// 16-aligned consecutive slots, and a row of 32 cells covers all 32 banks once, so
// the bank pair is fixed by the slot whatever the bin values are: the atomics of a
// step are free of bank conflicts by construction, not by chance as with the paper's
// 8-way interleave or its banked counters (App. A.1).  What skewed bin distributions
// (App. A.3) still cause is lanes of ONE instruction on the same address: the four rows
// of a wavefront that share a slot, when they share the bin too.  The LDS merges those
// at little cost (all 64 lanes on one cell: 8.5 instead of 6.4 cycles per instruction);
// measured on the whole kernel, a constant feature is 5 % and 60 % of the values in one
// bin 10 % slower than uniform bins at 64 bins, nothing at 256 bins -- against the 4x
// the paper reports for its hardware.  Switching the lanes of a frequent bin off does
// not help: an LDS atomic costs the same with 1 or 64 active lanes.
//
// Addressing.  The byte address of a cell inside its page is (bin << 8) | (8 *
// slot): one byte-permute builds it from the loaded bins and a per-lane table of
// the four values 8 * slot; the page is an immediate offset of the instruction.  With rows of 16 cells it is
// (bin >> 1) << 8 | (bin & 1) << 7 | (8 * slot): the lowest bits of a word's four bins first move into
// the table's bytes, four instructions more for four values.
//
// Arithmetic.  The paper adds floats with a compare-and-swap loop in local memory
// (App. B.3).  gfx950 has a native LDS float add, but it retires about 0.33
// lanes/clock/CU against about 10 for a 64-bit integer add, so values are
// accumulated as integers instead: rows are taken in epochs of kEpochRows = one row
// per thread.  A lane fetches the gradient and hessian of ITS row of the next epoch
// while the current epoch is accumulated; the workgroup sums their magnitudes, picks
// the largest power-of-two scales that cannot overflow a 27-bit field, and each lane
// quantises its own row once into a 64-bit addend that carries count, gradient and
// hessian.  The lanes that then work on a row fetch its addend with DPP moves, and
// every (row, feature) costs ONE 64-bit integer atomic.  After each epoch (kPairs:
// after every second one) the cells are drained into accumulators held in registers
// (each thread owns PP cells) and cleared.
// Error: each value is rounded once, by at most half a quantum; the quantum is at
// most sum|g|_epoch / (2^25 - 256), so a bin is off by at most 512 / (2^26 - 512) =
// 7.7e-6 of the leaf's sum |g| (likewise for h), and integer addition is
// order-independent.  (The accumulators add one fp32 rounding per epoch on top.)
//
// Memory.  The bins of a wavefront's 64 rows of an epoch sit in one register set of
// GPE row groups; as soon as a group has been added, the same group of the next
// epoch is requested into its registers; gradients / hessians are requested one
// epoch and row ids two epochs ahead, so that requests stay in flight across the
// epoch barriers and across the hand-out of work.
//
// All wavefronts of a workgroup share ONE histogram; no replica has to be reduced.
//
// chunk_stride: bytes from a lane-chunk of a row to the next: VEC, or more where the workgroup takes a part of every
// chunk only (plan_halves).
template <int CAP, int W, bool NIB, int NT, typename ACC, bool INDEXED, bool WIDE, bool SHORT>
__device__ __forceinline__ void build_tile(const uint8_t* __restrict__ tile, uint32_t row_stride, uint32_t chunk_stride,
                                           const int32_t* __restrict__ idx,
                                           const float* __restrict__ grad,
                                           const float* __restrict__ hess, bool stats_by_pos,
                                           uint32_t stat_shift, bool paced,
                                           uint32_t end,
                                           uint32_t first_unit, uint32_t first_epochs, uint32_t unit_epochs,
                                           uint32_t fixed_stride, uint32_t* counter,
                                           uint32_t counter_base, uint32_t n_firsts, unsigned long long* lds,
                                           uint32_t* __restrict__ out, const DirectOut& direct,
                                           uint32_t* __restrict__ out_lo = nullptr) {
  static_assert(!WIDE || sizeof(ACC) == 8, "wide cells are drained into fp64 accumulators");
  using S = TileShape<CAP, W, NIB, NT>;
  constexpr bool kShortRows = S::PITCH == 16;
  constexpr int NWORD = S::NWORD, LPR = S::LPR, RPW = S::RPW, NBW = S::NBW;
  constexpr int CELLS = S::CELLS, PP = S::PP, NW = S::NW;
  constexpr int NTBL = LPR == 8 ? 1 : 2;  // LPR 4: two byte-words share a page of 32 slots

  // Two epochs a drain.  With 256 bins a cell has two rows of an epoch, and draining its cells costs about as much as adding its
  // rows.  Wide cells have room for another epoch whatever the statistics are, as long as the two exponents are one apart
  // at most (wide_pair; what a row adds at the scale of the other epoch: wide_quantise).  The second epoch is counted in the
  // hessian cells, whose count field is free, so neither count passes 512.
  // (Root of 2,270,000 x 137 x 255 202 us drained after every epoch, 184 so, of 1,500,000 x 500 440 and 396; 60 % of the first as a
  // list 134 and 126; 64 leaves of all of the second 607 and 574.  With 64 or 16 bins, where a cell has more rows of an epoch,
  // it is between 4 % faster and 3 % slower.)
  constexpr bool kPairs = WIDE && CAP == 256;
  char* cells = reinterpret_cast<char*>(lds);
  constexpr int NCELLARR = WIDE ? 2 : 1;  // wide: gradient cells, then hessian cells
  float* red = reinterpret_cast<float*>(lds + NCELLARR * CELLS);  // [2 parities][2 stats][NW]
  uint32_t* unit_box = reinterpret_cast<uint32_t*>(red + 4 * NW);  // the unit just taken from the counter

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform, kept scalar
  const int j = lane % LPR;
  const int rho = lane / LPR;

  // Per-lane constants of the rotated step order.
  uint32_t sel[4];     // byte-permute selectors: byte 1 = bins byte q, byte 0 = table byte q
  uint32_t tbl[NTBL];  // 8 * slot-in-page of bytes q = 0..3
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t q = (uint32_t)(rho + k) & 3u;
    sel[k] = 0x0c0c0000u | ((4u + q) << 8) | q;
  }
#pragma unroll
  for (int v = 0; v < NTBL; ++v) {
    uint32_t t = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) t |= (uint32_t)(8 * (16 * v + j + LPR * q)) << (8 * q);
    tbl[v] = t;
  }

#pragma unroll
  for (int m = 0; m < PP * NCELLARR; ++m) lds[tid + m * NT] = 0ull;
  // The cells a thread drains: PP of one lane of slots.  Long leaves: cell t of thread t and every NT-th from there, so that a wavefront
  // takes 512 bytes of cells one after the other, 32 slots and 2 bins, and the wavefronts take turns in the bins; with 16 bins a thread
  // stays in one page instead (kernels of 4 pages spill less so: root of 3,000,000 x 400 x 16 238 us by thread, 229 so).  SHORT: a
  // wavefront takes 16 slots and 4 bins (16 cells in a row still cover all banks once) of bins of its own: a finished histogram leaves as
  // 48 bytes of a feature side by side and not 24, half as many lines a store, and the words of a partial block one after the other.
  // 128 leaves of half of 400,000 x 2,000 x 63 179 us with turns of 32 slots, 174 so; of 1,000,000 x 100 x 255 47.0 and 44.8; root of
  // 100,000 x 28 x 255, an epoch a workgroup, 22.3 with turns of 16, 18.7 so.  Long leaves are faster with turns: 1,500,000 x 500 x 255
  // 254 us, 259 with bins of a wavefront's own.
  constexpr bool kByThread = !SHORT && CAP != 16;
  constexpr int RUN = SHORT || S::PITCH == 16 ? 16 : 32, BINS = 64 / RUN;
  constexpr int RUNS = CELLS / (RUN * CAP);      // (those of a page without features among them)
  constexpr int WAVES = NW / RUNS;               // wavefronts of a run
  static_assert(kByThread || (NW % RUNS == 0 && CAP == BINS * WAVES * PP), "a thread drains cells of one slot");
  constexpr int kStepBins = SHORT ? BINS : BINS * WAVES;  // from a thread's bin to its next
  const int first_slot = wave % RUNS * RUN, first_bin = wave / RUNS * (SHORT ? BINS * PP : BINS);
  const int run_cell = first_slot / S::PITCH * (CAP * S::PITCH) + first_slot % S::PITCH + first_bin * S::PITCH;  // scalar
  auto owned_cell = [&](int t) {  // of thread t, the first one
    return kByThread ? t : run_cell + (t & 63) / RUN * S::PITCH + (t & 63) % RUN;
  };
  constexpr int kOwnedStep = kByThread ? NT : kStepBins * S::PITCH;  // ... to the next
  ACC acc_g[PP], acc_h[PP];
  uint32_t acc_c[PP];
#pragma unroll
  for (int m = 0; m < PP; ++m) {
    acc_g[m] = (ACC)0;
    acc_h[m] = (ACC)0;
    acc_c[m] = 0u;
  }

  static_assert(NW == 8, "the wave sums of one statistic fill one group of 8 lanes");
  auto reduce_abs = [&](float ag, float ah, int parity) {
    ag = wave_sum_to_lane63(ag);
    ah = wave_sum_to_lane63(ah);
    if (lane == 63) {
      red[parity * 2 * NW + wave] = ag;
      red[parity * 2 * NW + NW + wave] = ah;
    }
  };
  // lanes 0..7 fetch the wave sums of |g|, lanes 8..15 those of |h|; the two totals are
  // moved to scalar registers and turned into exponents there
  auto request_scales = [&](int parity, int lane) { return red[parity * 2 * NW + (lane & (2 * NW - 1))]; };
  auto scales_from = [&](float v, int& kg, int& kh) {
    v = sum_in_8(v) * 1.001953125f;
    const uint32_t bits_g = (uint32_t)__builtin_amdgcn_readlane(__float_as_uint(v), 0);
    const uint32_t bits_h = (uint32_t)__builtin_amdgcn_readlane(__float_as_uint(v), 8);
    kg = epoch_scale_exp(bits_g);
    kh = epoch_scale_exp(bits_h);
  };

  // Row ownership.  In every epoch the wavefront takes 64 consecutive leaf positions,
  // as GPE row groups of RPW rows; lane (rho, j) works on row rho of every group and
  // OWNS (fetches the row id, gradient and hessian of, and quantises) row rho of
  // group j.  The owner of a row therefore sits among the LPR lanes that work on it,
  // and its values reach them with DPP broadcasts, without LDS traffic.
  static_assert(S::GPE == LPR, "one owner lane per (row, group)");
  const uint32_t own = (uint32_t)wave * 64u + (uint32_t)(j * RPW + rho);
  // leaf position (clamped to the chunk's last row, so that every load stays in
  // range), validity and row id of the row this lane owns in the epoch starting at e0
  auto own_pos = [&](uint32_t e0) {
    const uint32_t i = e0 + own;
    return i < end ? i : end - 1;
  };
  auto own_valid = [&](uint32_t e0) { return e0 + own < end; };
  auto load_row_id = [&](uint32_t e0) -> uint32_t {
    const uint32_t i = own_pos(e0);
    return INDEXED ? (uint32_t)*reinterpret_cast<const int32_t*>(
                         reinterpret_cast<const char*>(idx) + (i << 2))
                   : i;
  };
  auto load_stat = [&](const float* a, uint32_t r) {
    return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(a) + (r << stat_shift));
  };
  // value of `v` held by the owner of this lane's row of group gi: lane j = gi of the
  // LPR lanes that share the row
  auto from_owner = [&](uint32_t v, auto gi_tag) -> uint32_t {
    constexpr int gi = decltype(gi_tag)::value;
    if (LPR == 4) {  // quad broadcast: every lane of a quad takes lane gi of the quad
      return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, gi * 0x55, 0xf, 0xf, false);
    }
    // LPR 8: lanes 0..7 of each row of 16 take lane gi, lanes 8..15 take lane 8 + gi
    const int lo8 = __builtin_amdgcn_mov_dpp((int)v, 0x150 + gi, 0xf, 0xf, false);
    return (uint32_t)__builtin_amdgcn_update_dpp(lo8, (int)v, 0x158 + gi, 0xf, 0xc, false);
  };

  // Bins of one row group.  Without an index list the rows of an epoch are
  // consecutive, so group gi sits gi * RPW rows behind group 0 (added to the uniform
  // base) and rows past the chunk end are simply read: they lie inside
  // the matrix, its slack or the columns behind it, and their addend is zero.  With an index list the
  // row's byte offset (`rows`) comes from the row's owner.
  constexpr int GPE = S::GPE;
  auto load_group = [&](uint4& w, uint32_t rows, uint32_t off0, auto gi_tag) {
    constexpr int gi = decltype(gi_tag)::value;
    uint32_t off;  // 32-bit byte offsets ((n_rows + slack) * row_stride < 2^32)
    const uint8_t* base = tile;
    if (INDEXED) {
      off = from_owner(rows, gi_tag) + chunk_stride * (uint32_t)j;
    } else {
      off = off0;
      base += (uint32_t)(gi * RPW) * row_stride;
    }
    if (NWORD == 4) {
      w = *reinterpret_cast<const uint4*>(base + off);
    } else if (NWORD == 2) {
      const uint2 v = *reinterpret_cast<const uint2*>(base + off);
      w.x = v.x;
      w.y = v.y;
    } else {
      w.x = *reinterpret_cast<const uint32_t*>(base + off);
    }
  };
  // lo, hi: the addend of the row this lane owns (zero for a row past the chunk end); wide:
  // the gradient cell's addend, and lo2, hi2 the hessian cell's
  auto add_group = [&](const uint4& w, uint32_t lo, uint32_t hi, uint32_t lo2, uint32_t hi2, auto gi_tag) {
    const unsigned long long add =
        ((unsigned long long)from_owner(hi, gi_tag) << 32) | from_owner(lo, gi_tag);
    unsigned long long add2 = 0ull;
    if (WIDE) add2 = ((unsigned long long)from_owner(hi2, gi_tag) << 32) | from_owner(lo2, gi_tag);
    uint32_t bword[NBW];
#pragma unroll
    for (int x = 0; x < NWORD; ++x) {
      const uint32_t word = x == 0 ? w.x : (x == 1 ? w.y : (x == 2 ? w.z : w.w));
      if (NIB) {
        bword[2 * x] = word & 0x0f0f0f0fu;
        bword[2 * x + 1] = (word >> 4) & 0x0f0f0f0fu;
      } else {
        bword[x] = word;  // the pack kernel keeps every bin value below CAP
      }
    }
#pragma unroll
    for (int bw = 0; bw < NBW; ++bw) {
      const int page = LPR == 8 ? bw : (bw >> 1);
      const int tv = LPR == 8 ? 0 : (bw & 1);
      const uint32_t upper = kShortRows ? (bword[bw] >> 1) & 0x7f7f7f7fu : bword[bw];
      const uint32_t lower = kShortRows ? ((bword[bw] << 7) & 0x80808080u) | tbl[tv] : tbl[tv];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t a = __builtin_amdgcn_perm(upper, lower, sel[k]);
        __hip_atomic_fetch_add(
            reinterpret_cast<unsigned long long*>(cells + a + page * (CAP * 256)), add,
            __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (WIDE) {
          __hip_atomic_fetch_add(
              reinterpret_cast<unsigned long long*>(cells + a + page * (CAP * 256) + CELLS * 8), add2,
              __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
      }
    }
  };
  static_assert(GPE == 4 || GPE == 8, "row groups per epoch");
  // (an epoch past the leaf is read at the leaf's last epoch: in range, and ignored)
  const uint32_t n_epochs_leaf = (end + kEpochRows - 1) / kEpochRows;
  const uint32_t past = n_epochs_leaf * (uint32_t)kEpochRows;  // position of "no epoch"
  const uint32_t lane_offset = (uint32_t)rho * row_stride + chunk_stride * (uint32_t)j;
  auto group_offset0 = [&](uint32_t e0) {
    const uint32_t e = e0 < past ? e0 : past - (uint32_t)kEpochRows;
    return (e + (uint32_t)wave * 64u) * row_stride + lane_offset;
  };
  // The bins of all row groups of one epoch, requested in group order.  (The scheduling
  // barriers keep that order: the epoch loop waits for group gi with "at most GPE + 1
  // younger requests outstanding", which is only right when the first epoch's requests were
  // issued in the order the loop re-issues them.)
  auto load_epoch = [&](uint4 (&w)[GPE], uint32_t rows, uint32_t e0) {
    const uint32_t off0 = group_offset0(e0);
    const uint32_t row_off = rows * row_stride;
    auto step = [&](auto gi_tag) {
      constexpr int gi = decltype(gi_tag)::value;
      load_group(w[gi], row_off, off0, gi_tag);
      __builtin_amdgcn_sched_barrier(0);
    };
    step(std::integral_constant<int, 0>{});
    step(std::integral_constant<int, 1>{});
    step(std::integral_constant<int, 2>{});
    step(std::integral_constant<int, 3>{});
    if constexpr (GPE == 8) {
      step(std::integral_constant<int, 4>{});
      step(std::integral_constant<int, 5>{});
      step(std::integral_constant<int, 6>{});
      step(std::integral_constant<int, 7>{});
    }
  };
  // Takes the sums of a cell out of local memory (read and clear in one operation) ...
  auto request_cell = [&](int i) {
    return __hip_atomic_exchange(&lds[i], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  // ... and adds them to this thread's accumulators of its cell m (wide: th = the hessian cell).
  auto drain_cell = [&](int m, unsigned long long t, unsigned long long th, float inv_g, float inv_h,
                        double inv_gw, double inv_hw) {
    if constexpr (kPairs) {
      const uint32_t lo = (uint32_t)t, lo_h = (uint32_t)th;
      acc_c[m] += (lo & ((1u << kCountBits) - 1u)) + (lo_h & ((1u << kCountBits) - 1u));
      acc_g[m] = (ACC)add_wide_sum((double)acc_g[m], lo, (uint32_t)(t >> 32), inv_gw);
      acc_h[m] = (ACC)add_wide_sum((double)acc_h[m], lo_h, (uint32_t)(th >> 32), inv_hw);
      return;
    }
    if constexpr (WIDE) {
      // the count sits below the gradient sum; an arithmetic shift drops it whatever the sign
      acc_c[m] += (uint32_t)t & ((1u << kCountBits) - 1u);
      acc_g[m] = (ACC)fma(i64_to_f64((long long)t >> kCountBits), inv_gw, (double)acc_g[m]);
      acc_h[m] = (ACC)fma(i64_to_f64((long long)th >> kCountBits), inv_hw, (double)acc_h[m]);
      return;
    }
    // both sums times 2^kSumPad (the scales inv_g, inv_h allow for it)
    const CellSums sums = cell_sums((uint32_t)t, (uint32_t)(t >> 32));
    const int32_t gs = sums.grad, hs = sums.hess;
    const uint32_t c = sums.count;
    // integer * power of two + accumulator, rounded once
    if (sizeof(ACC) == 8) {
      acc_g[m] = (ACC)fma((double)gs, (double)inv_g, (double)acc_g[m]);
      acc_h[m] = (ACC)fma((double)hs, (double)inv_h, (double)acc_h[m]);
    } else {
      acc_g[m] = (ACC)__fmaf_rn((float)gs, inv_g, (float)acc_g[m]);
      acc_h[m] = (ACC)__fmaf_rn((float)hs, inv_h, (float)acc_h[m]);
    }
    acc_c[m] += c;
  };
  // Adds the row groups of one epoch and, as soon as a group's registers are free,
  // requests the same group of the next epoch into them: every request has a whole
  // epoch to complete, requests are spread evenly over the epoch, and one register set
  // serves both epochs.
  auto add_and_reload = [&](uint4 (&w)[GPE], uint32_t lo, uint32_t hi, uint32_t lo2, uint32_t hi2,
                            uint32_t rows_nxt, uint32_t e0_nxt) {
    const uint32_t off0 = group_offset0(e0_nxt);
    const uint32_t row_off = rows_nxt * row_stride;
    auto step = [&](auto gi_tag) {
      constexpr int gi = decltype(gi_tag)::value;
      add_group(w[gi], lo, hi, lo2, hi2, gi_tag);
      load_group(w[gi], row_off, off0, gi_tag);
    };
    step(std::integral_constant<int, 0>{});
    step(std::integral_constant<int, 1>{});
    step(std::integral_constant<int, 2>{});
    step(std::integral_constant<int, 3>{});
    if constexpr (GPE == 8) {
      step(std::integral_constant<int, 4>{});
      step(std::integral_constant<int, 5>{});
      step(std::integral_constant<int, 6>{});
      step(std::integral_constant<int, 7>{});
    }
  };

  // Work distribution.  The workgroups of a tile share out the n_epochs epochs of the
  // leaf in units of consecutive epochs: the first n_firsts units have first_epochs each, the others
  // unit_epochs.  Workgroup c of the tile starts with unit c; in a unit's third-last epoch one lane takes the
  // next one from the tile's counter (a global atomic that starts at zero: the take is counter_base + its old
  // value, counter_base = the units the workgroups started with), and the pipeline of
  // requests (row ids two epochs ahead, gradients / hessians and bins one epoch ahead)
  // runs on from the last epoch of a unit into the first epoch of the next.  Fast and
  // slow workgroups (the CU issues the instructions of its oldest workgroup first) so
  // end within a unit of each other, and one partial block per workgroup suffices.
  // Looking two epochs ahead needs the next unit from a unit's second-last epoch on:
  // the counter is only used with units of at least 3 epochs; shorter units (short
  // leaves) are handed out one per workgroup, in a fixed stride.
  // With fixed_stride != 0 the counter is not used: after unit u a workgroup takes unit
  // u + fixed_stride.  The grouping of epochs into partial sums is then the same in
  // every run, and so is every bit of the result.
  struct Pos {
    uint32_t row;   // first leaf position of the epoch; `past`: no epoch
    uint32_t left;  // epochs of its unit from here on
    uint32_t unit;
  };
  const uint32_t n_first = n_firsts * first_epochs;  // epochs in the long first units
  const uint32_t n_units = n_first >= n_epochs_leaf
                               ? n_firsts : n_firsts + (n_epochs_leaf - n_first + unit_epochs - 1) / unit_epochs;
  uint32_t next_unit = n_units;  // the unit taken from the counter (n_units or more: none)
  auto unit_first = [&](uint32_t u) {
    Pos r;
    const uint32_t e = u < n_firsts ? u * first_epochs : n_first + (u - n_firsts) * unit_epochs;
    r.row = u < n_units && e < n_epochs_leaf ? e * (uint32_t)kEpochRows : past;
    r.left = u < n_firsts ? first_epochs : unit_epochs;
    r.unit = u;
    return r;
  };
  auto after = [&](Pos x) {  // the epoch after x in this workgroup's sequence
    if (x.row >= past) return x;
    Pos r;
    r.row = x.row + kEpochRows;
    r.left = x.left - 1;
    r.unit = x.unit;
    // the leaf may end inside its last unit
    if (r.left == 0 || r.row >= past) {
      // The taken unit is used up: until the next take arrives there is no further unit
      // (only the leaf's short last unit can end before that, and nothing follows it).
      r = unit_first(fixed_stride ? x.unit + fixed_stride : next_unit);
      next_unit = n_units;
    }
    return r;
  };
  Pos p0 = unit_first(first_unit), p1 = after(p0), p2 = after(p1);

  int kg, kh;
  // rows the lane owns in the current epoch and the next one; the current row's stats
  uint32_t row_cur = load_row_id(p0.row);
  uint32_t row_nxt = load_row_id(p1.row);
  // gradients / hessians are indexed by row id, or (stats_by_pos) by leaf position when the
  // call has gathered them into leaf order beforehand
  float g_cur = load_stat(grad, stats_by_pos ? own_pos(p0.row) : row_cur);
  float h_cur = load_stat(hess, stats_by_pos ? own_pos(p0.row) : row_cur);
  uint4 w[GPE];
  load_epoch(w, row_cur, p0.row);
  {
    const bool ok = own_valid(p0.row);
    reduce_abs(ok ? fabsf(g_cur) : 0.0f, ok ? fabsf(h_cur) : 0.0f, 0);
  }
  __syncthreads();  // also orders the LDS clearing before the first atomics
  scales_from(request_scales(0, lane), kg, kh);

  // The row that a lane owns -> what it adds to its cells (cell_format.h; wide: 1 + gq * 2^10 to the gradient cell, hq * 2^10 to
  // the hessian cell); ok: there is such a row.
  struct Addend {
    uint32_t lo, hi, lo2, hi2;
  };
  auto wide_exp = [](int k) { return wide_cell_exp(k, kPairs); };
  // second: of two epochs a drain; coarse_g, coarse_h: and its own exponent is one less (wide_quantise)
  auto quantise = [&](bool ok, bool second, int coarse_g, int coarse_h) {
    Addend a = {0u, 0u, 0u, 0u};
    if constexpr (WIDE) {
      const long long gq = wide_quantise(g_cur, wide_exp(kg), coarse_g), hq = wide_quantise(h_cur, wide_exp(kh), coarse_h);
      const unsigned long long ag = ((unsigned long long)gq << kCountBits) + (kPairs && second ? 0ull : 1ull);
      const unsigned long long ah = ((unsigned long long)hq << kCountBits) + (kPairs && second ? 1ull : 0ull);
      a.lo = ok ? (uint32_t)ag : 0u;
      a.hi = ok ? (uint32_t)(ag >> 32) : 0u;
      a.lo2 = ok ? (uint32_t)ah : 0u;
      a.hi2 = ok ? (uint32_t)(ah >> 32) : 0u;
    } else {
      const CellWords add = cell_addend(__float2int_rn(g_cur * pow2f(kg)), __float2int_rn(h_cur * pow2f(kh)));
      a.lo = ok ? add.lo : 0u;
      a.hi = ok ? add.hi : 0u;
    }
    return a;
  };
  // The integer sums of an epoch -> registers, and the cells cleared for the next one.  All requests leave before the first
  // answer is waited for, those that `first` makes first of all: answers come back in order, so the cells are then decoded one by
  // one as they arrive.  (The scheduling barrier keeps the arithmetic of `second` from being waited for between the requests.)
  auto drain = [&](auto&& first, auto&& second) {
    const float inv_g = pow2f(-kg) * (1.0f / (1 << kSumPad)), inv_h = pow2f(-kh) * (1.0f / (1 << kSumPad));
    // (of sums, or of whole cells)
    const double inv_gw = pow2d(-wide_exp(kg) - (kPairs ? kCountBits : 0)), inv_hw = pow2d(-wide_exp(kh) - (kPairs ? kCountBits : 0));
    if (WIDE && !kPairs && (kg <= kWidePastExp || kh <= kWidePastExp)) {
      // kWidePastExp: rare, so here, cell by cell (the registers are taken), and what follows then finds empty cells.  (As the
      // other branch of what follows it costs all wide kernels 10 to 40 registers.)
#pragma unroll
      for (int m = 0; m < PP; ++m) {
        const int at = owned_cell(tid) + m * kOwnedStep;
        const unsigned long long t = request_cell(at), th = request_cell((WIDE ? CELLS : 0) + at);
        acc_c[m] += (uint32_t)t & ((1u << kCountBits) - 1u);
        acc_g[m] = (ACC)fma((double)((long long)t >> kCountBits), inv_gw, (double)acc_g[m]);
        acc_h[m] = (ACC)fma((double)((long long)th >> kCountBits), inv_hw, (double)acc_h[m]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // The 16-bin variant has 64 registers (8 wavefronts a SIMD) and no room for addresses that are only used here: kept, they
    // are spilled, and reading them back waits for everything requested before, all of the next epoch's bins.  Formed here
    // anew (32 leaves of half of 2,000,000 x 150 x 16 53.8 -> 49.4 us, 25 % of the rows 47.0 -> 44.4).
    int drain_tid = tid;
    if constexpr (CAP == 16 && !WIDE) {
      int l;
      asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
      drain_tid = wave * 64 + l;
    }
    const int drain_cell0 = owned_cell(drain_tid);
    first(drain_tid);
    unsigned long long cell[PP], cell_h[WIDE ? PP : 1];
#pragma unroll
    for (int m = 0; m < PP; ++m) {
      cell[m] = request_cell(drain_cell0 + m * kOwnedStep);
      if constexpr (WIDE) cell_h[m] = request_cell(CELLS + drain_cell0 + m * kOwnedStep);
    }
    __builtin_amdgcn_sched_barrier(0);
    second();
#pragma unroll
    for (int m = 0; m < PP; ++m) drain_cell(m, cell[m], cell_h[WIDE ? m : 0], inv_g, inv_h, inv_gw, inv_hw);
  };

  uint32_t parity = 0;
  uint32_t row_nn = 0u;
  float g_nxt = 0.0f, h_nxt = 0.0f;
  // Whether the leaf's last epoch, where rows may be missing, has code of its own (below).  Long leaves, to which it is nothing, are
  // a little faster with one loop: 2,270,000 x 137 x 255 124.0 us, 125.2 with two; 1,500,000 x 330 x 64 with wide sums 215 and 219.
  constexpr bool kLastApart = SHORT || kPairs;
  // An epoch of 512 rows: requests for later ones, its additions, and the sums of the next.  Returns whether a unit was taken.
  auto add_epoch = [&](bool second, int coarse_g, int coarse_h) {
    const bool takes = !fixed_stride && p0.left == 3;
    uint32_t taken = 0;
    if (takes && tid == 0)
      taken = counter_base + __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // ---- requests for later epochs
    row_nn = load_row_id(p2.row);
    const uint32_t stat_nxt = stats_by_pos ? own_pos(p1.row) : row_nxt;
    g_nxt = load_stat(grad, stat_nxt);
    h_nxt = load_stat(hess, stat_nxt);
    const Addend add = quantise(kLastApart || own_valid(p0.row), second, coarse_g, coarse_h);
    // The atomics are what the kernel is bound by; the drain of a co-resident workgroup is
    // mostly VALU work.  Raised priority lets the waves that feed the LDS pipe issue first,
    // and the other workgroup's drain fills the gaps (8-12 % on the 256-bin variants).
    __builtin_amdgcn_s_setprio(1);
    add_and_reload(w, add.lo, add.hi, add.lo2, add.hi2, row_nxt, p1.row);
    __builtin_amdgcn_s_setprio(0);

    parity ^= 1u;
    {
      const bool ok = own_valid(p1.row);
      reduce_abs(ok ? fabsf(g_nxt) : 0.0f, ok ? fabsf(h_nxt) : 0.0f, (int)parity);
    }
    if (takes && tid == 0) unit_box[0] = taken;
    // Workgroups that share cache lines (tile_plan.h) drift apart if nothing holds them together, and a
    // line is then fetched twice.  Waiting here for half of the next epoch's bins lets a workgroup that runs
    // ahead, whose requests miss, be caught up by the one whose requests hit.  (First pass over the rows of
    // 2,000,000 x 500 x 64 283 us with and 318 without, of 400,000 x 2,000 x 63 234 and 250; waiting for all of the next
    // epoch's bins instead 287 and 239.  32-byte tiles do not wait: a workgroup spends longer on an epoch there, in the
    // drain, and roots are the same either way (192.1 and 192.0 us for 1,000,000 x 500 x 255), but half and a quarter
    // of the rows go from 119 / 76 to 125 / 80 us with the wait.  A remainder does beside the one tile whose lines it shares:
    // it has half the cells to drain and runs ahead, two leaves of all of 4,000,000 x 33 x 255 108 us with the wait and 120
    // without, four 108 and 121; 64 leaves of 48 features 168 and 164.)
    if (paced) __builtin_amdgcn_s_waitcnt(GPE == 8 ? 0x0f74 : 0x0f72);  // vmcnt(GPE / 2)
    __syncthreads();  // all atomics of the epoch have landed
    return takes;
  };
  auto to_next_epoch = [&] {
    p0 = p1;
    p1 = p2;
    p2 = after(p2);
    row_cur = row_nxt;
    row_nxt = row_nn;
    g_cur = g_nxt;
    h_cur = h_nxt;
  };
  while (p0.row + (kLastApart ? (uint32_t)kEpochRows - 1u : 0u) < end) {  // uniform over the workgroup
    bool takes = add_epoch(false, 0, 0);
    if constexpr (kPairs) {
      if (p1.row + (uint32_t)kEpochRows <= end) {
        int kg_nxt, kh_nxt;
        scales_from(request_scales((int)parity, lane), kg_nxt, kh_nxt);
        if (wide_pair(kg, kg_nxt) && wide_pair(kh, kh_nxt)) {
          // (no barrier: `red` has another place for the next epoch, and units are taken three epochs apart at least)
          if (takes) next_unit = __builtin_amdgcn_readfirstlane(unit_box[0]);
          to_next_epoch();
          takes = add_epoch(true, kg_nxt < kg, kh_nxt < kh);
        }
      }
    }
    float next_sums = 0.0f;
    uint32_t box = 0u;
    int kg_nxt = 0, kh_nxt = 0;
    drain(
        [&](int drain_tid) {
          next_sums = request_scales((int)parity, drain_tid);
          box = unit_box[0];
        },
        [&] {
          scales_from(next_sums, kg_nxt, kh_nxt);
          if (takes) next_unit = __builtin_amdgcn_readfirstlane(box);
        });
    kg = kg_nxt;
    kh = kh_nxt;
    to_next_epoch();
    __syncthreads();  // cells are clear, `red` and the unit box are read, before reuse
  }
  // The leaf's last epoch, where rows are missing: nothing follows it, and wavefronts without a row add nothing.  (As one more
  // turn of the loop, which adds zeros and requests rows that nobody takes: 128 leaves of half of 400,000 x 2,000 x 63 174 us, 162
  // so; 64 equal leaves of 1,500,000 x 500 x 255, 46 epochs a workgroup, 371 and 353 (with the drains of then; unequal leaves, of which the
  // longest count, gain nothing); 32 of half of 100,000 x 50 x 64 15.9 and 14.3.  A branch around the additions inside the loop makes
  // every turn wait for all requests: root of 10,500,000 x 28 x 255 127 us, 146 so.)
  if (kLastApart && p0.row < end) {
    const Addend add = quantise(own_valid(p0.row), false, 0, 0);
    if (p0.row + (uint32_t)wave * 64u < end) {
      auto step = [&](auto gi_tag) {
        add_group(w[decltype(gi_tag)::value], add.lo, add.hi, add.lo2, add.hi2, gi_tag);
      };
      step(std::integral_constant<int, 0>{});
      step(std::integral_constant<int, 1>{});
      step(std::integral_constant<int, 2>{});
      step(std::integral_constant<int, 3>{});
      if constexpr (GPE == 8) {
        step(std::integral_constant<int, 4>{});
        step(std::integral_constant<int, 5>{});
        step(std::integral_constant<int, 6>{});
        step(std::integral_constant<int, 7>{});
      }
    }
    __syncthreads();  // all atomics have landed
    drain([](int) {}, [] {});
  }

  if (direct.hist) {
    // The tile's only workgroup: its sums are the histogram.  Cell -> (bin, slot) ->
    // feature, as the reduction pass would do it.
    TilePlan plan;
    plan.cap = CAP;
    plan.nib = NIB ? 1 : 0;
    plan.wm = direct.wm;
    plan.n_main = direct.n_main;
    plan.wr = direct.wr;
    plan.row_bytes = plan.feat_bytes = 0;  // not used by the slot -> feature map
    if constexpr (kByThread) {
      // (Rarely taken: a matrix of more tiles than workgroups that fit the machine.  What is shared by a thread's cells stays
      // unshared, because the loop above is laid out worse otherwise: 1,500,000 x 500 x 255 258 us, 262 written as below.)
#pragma unroll
      for (int m = 0; m < PP; ++m) {
        const int cell = tid + m * NT;
        const int bin = cell / S::PITCH % CAP, slot = cell / (CAP * S::PITCH) * S::PITCH + cell % S::PITCH;
        const int32_t f = plan_feature_of(plan, direct.tile, direct.first_slot + slot);
        if (slot < S::SLOTS && bin < direct.n_bins && f < direct.n_features) {
          gbdt_bin_t r;
          r.grad = (float)acc_g[m];
          r.hess = (float)acc_h[m];
          r.count = acc_c[m];
          direct.hist[(size_t)f * direct.n_bins + bin] = r;
        }
      }
      return;
    }
    const int slot = first_slot + lane % RUN, bin0 = first_bin + lane / RUN;
    const int32_t f = plan_feature_of(plan, direct.tile, direct.first_slot + slot);
    if (slot < S::SLOTS && f < direct.n_features) {
      gbdt_bin_t* to = direct.hist + (size_t)f * direct.n_bins;
#pragma unroll
      for (int m = 0; m < PP; ++m) {
        const int bin = bin0 + kStepBins * m;
        if (bin < direct.n_bins) {
          gbdt_bin_t r;
          r.grad = (float)acc_g[m];
          r.hess = (float)acc_h[m];
          r.count = acc_c[m];
          to[bin] = r;
        }
      }
    }
    return;
  }
  // partial block layout: [stat][cell] words
  const int cell0 = owned_cell(tid);
#pragma unroll
  for (int m = 0; m < PP; ++m) {
    out[cell0 + m * kOwnedStep] = __float_as_uint((float)acc_g[m]);
    out[CELLS + cell0 + m * kOwnedStep] = __float_as_uint((float)acc_h[m]);
    out[2 * CELLS + cell0 + m * kOwnedStep] = acc_c[m];
  }
  if constexpr (WIDE) {
    // what fp32 cannot hold of the fp64 sums goes into a second block of the same layout (count
    // 0), which the reduction pass adds like any other workgroup's
#pragma unroll
    for (int m = 0; m < PP; ++m) {
      const double g = (double)acc_g[m], h = (double)acc_h[m];
      out_lo[cell0 + m * kOwnedStep] = __float_as_uint((float)(g - (double)(float)g));
      out_lo[CELLS + cell0 + m * kOwnedStep] = __float_as_uint((float)(h - (double)(float)h));
      out_lo[2 * CELLS + cell0 + m * kOwnedStep] = 0u;
    }
  }
}

// Words of one partial block of a tile of width W.
template <int CAP, int W, bool NIB, int NT>
__device__ __host__ constexpr int block_words() {
  return 3 * TileShape<CAP, W, NIB, NT>::CELLS;
}

// Work is split by feature tiles and by samples (Sec. 4, "Parallel By Features and
// Data"): every tile has a fixed set of workgroups that share out its epochs.  Block
// -> (tile, workgroup of the tile) by line_block (batch_plan.h): tiles that share lines of the
// matrix on one XCD, otherwise neighbouring blocks on different tiles; either way the workgroups of a column start
// together, and the row ids / gradients / hessians of an epoch are fetched from HBM once and served to the
// other tiles from cache.
template <int CAP, int WM, bool NIB, int NT, bool WIDE, bool HALVES>
struct BuildShape {
  static_assert(!HALVES || (WIDE && CAP == 256), "see plan_halves");
  static constexpr bool kHalves = HALVES;
  static constexpr int kMainW = kHalves ? 16 : WM;        // width of the tile that a workgroup has the cells of
  static constexpr int kCells = (WIDE ? 2 : 1) * TileShape<CAP, kMainW, NIB, NT>::CELLS;
  // the cells (8 bytes each; two histograms with wide accumulation), the reduction scratch and the unit box
  static constexpr int kLdsWords = kCells + (4 * (NT / 64) * 4 + 7) / 8 + 1;
};

// One workgroup's work on (tile, half) of a leaf: build_tile with the tile's width.  leaf_out: the leaf's partial blocks,
// `chunks` of every part (tile or half), parts back to back, wg the workgroup's among them; with wide accumulation its second
// block lies wgs blocks behind its first.
template <int CAP, int WM, bool NIB, int NT, typename ACC, bool INDEXED, bool WIDE, bool HALVES, bool SHORT, typename... REST>
__device__ __forceinline__ void build_part(const uint8_t* packed, int64_t n_rows, int32_t n_main, int32_t wr,
                                           int32_t line_tiles, int32_t t, int32_t half, uint32_t* leaf_out, size_t chunks,
                                           size_t wg, size_t wgs, gbdt_bin_t* direct_hist, int32_t n_features,
                                           int32_t n_bins, unsigned long long* lds, const int32_t* idx, const float* grad,
                                           const float* hess, bool by_pos, uint32_t stat_shift, REST... rest) {
  using BS = BuildShape<CAP, WM, NIB, NT, WIDE, HALVES>;
  const TileAt at = plan_tile_at(WM, n_main, wr, n_rows, line_tiles, t);
  const uint8_t* tile = packed + at.off;
  const uint32_t stride = (uint32_t)at.stride;
  const bool paced = WM == 64 && at.shared;  // (see the wait in build_tile)
  const DirectOut direct = {direct_hist, t, WM, n_main, wr, 16 * half, n_features, n_bins};
  constexpr size_t kMainBlock = (size_t)block_words<CAP, BS::kMainW, NIB, NT>();
  if (t < n_main) {
    constexpr uint32_t kVec = TileShape<CAP, WM, NIB, NT>::VEC;
    const size_t part = BS::kHalves ? 2 * (size_t)t + (size_t)half : (size_t)t;
    uint32_t* out = leaf_out + (part * chunks + wg) * kMainBlock;
    build_tile<CAP, BS::kMainW, NIB, NT, ACC, INDEXED, WIDE, SHORT>(tile + 4 * half, stride, kVec, idx, grad, hess, by_pos, stat_shift,
                                                             paced, rest..., lds, out, direct, out + wgs * kMainBlock);
    return;
  }
  uint32_t* rem_base = leaf_out + (size_t)(BS::kHalves ? 2 * n_main : n_main) * chunks * kMainBlock;
  auto remainder = [&](auto width) {
    constexpr int W = decltype(width)::value;
    constexpr size_t kBlock = (size_t)block_words<CAP, W, NIB, NT>();
    build_tile<CAP, W, NIB, NT, ACC, INDEXED, WIDE, SHORT>(tile, stride, TileShape<CAP, W, NIB, NT>::VEC, idx, grad, hess, by_pos,
                                                    stat_shift, paced || (!WIDE && WM == 32 && n_main == 1 && at.shared),
                                                    rest..., lds, rem_base + wg * kBlock, direct,
                                                    rem_base + (wgs + wg) * kBlock);
  };
  if (wr == 16) {
    remainder(std::integral_constant<int, 16>{});
  } else if constexpr (WM > 32) {
    remainder(std::integral_constant<int, 32>{});
  }
}

// SHORT: for leaves whose end is much of a workgroup's work (leaf_is_short, batch_is_short; what differs: build_tile).
template <int CAP, int WM, bool NIB, int NT, int WPE, typename ACC, bool INDEXED, bool WIDE = false, bool HALVES = false,
          bool SHORT = false>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(WPE, WPE)))
hist_build_kernel(BuildArgs a) {
  using BS = BuildShape<CAP, WM, NIB, NT, WIDE, HALVES>;
  __shared__ __align__(16) unsigned long long lds[BS::kLdsWords];
  int32_t t, half = 0, c;  // c: workgroup of the tile
  if constexpr (BS::kHalves) {
    const HalfBlock hb = half_block(WM, a.n_main, a.deal, (uint32_t)a.wgs, false, blockIdx.x);
    t = hb.tile;
    half = hb.half;
    c = (int32_t)hb.col;
  } else {
    const LineBlock lb = line_block(WM, a.n_main, a.wr, a.deal, (uint32_t)a.wgs, false, blockIdx.x);
    t = lb.tile;
    c = (int32_t)lb.col;
  }
  uint32_t* counter = a.counters + plan_counter_slot(BS::kHalves ? 2 * t + half : t);
  const uint32_t n_firsts = a.first_epochs ? (uint32_t)a.wgs : 0u;
  build_part<CAP, WM, NIB, NT, ACC, INDEXED, WIDE, HALVES, SHORT>(
      a.packed, a.n_rows, a.n_main, a.wr, a.line_tiles, t, half, a.partials, (size_t)a.chunks, (size_t)c, (size_t)a.wgs,
      a.direct_out, a.n_features, a.n_bins, lds, a.idx, a.grad, a.hess, a.stats_by_pos != 0, 2u, (uint32_t)a.n_leaf,
      (uint32_t)c, (uint32_t)a.first_epochs, (uint32_t)a.unit_epochs, (uint32_t)a.fixed_stride, counter, (uint32_t)a.wgs,
      n_firsts);
}

// Gradients and hessians of a row list, in list order: g_out[i] = grad[idx[i]].  The paper
// has the CPU prepare these "ordered" arrays for every leaf (App. A.5, App. C.1); here they pay
// when many feature tiles would each gather the same scattered 4-byte values again.
__global__ void __launch_bounds__(256)
stats_gather_kernel(const int32_t* __restrict__ idx, const float* __restrict__ grad,
                    const float* __restrict__ hess, int64_t n, float* __restrict__ g_out,
                    float* __restrict__ h_out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint32_t r = (uint32_t)idx[i];
  g_out[i] = grad[r];
  h_out[i] = hess[r];
}

// The same for several row lists, dealt out to the XCDs by parts of the lists: an XCD takes the k-th eighth of every
// list, one list after the other.  Lists of a tree's leaves ascend, so those are about the same rows of grad and hess, whose
// lines the XCD's L2 then fetches once for all lists instead of once for each (64 leaves of 1,500,000 rows: 30 us in list
// order, 18 so).  Any other lists are gathered as well.  A block takes kGatherRows positions of a part.  Lists are
// segments of idx; what belongs to position i of idx goes to position i of the output, or i - wrap from `wrap` on (the two row
// buffers of a tree share one set of positions).
constexpr int kGatherLists = 300;
constexpr int kGatherRows = 1024;
struct GatherTable {
  uint32_t first[kGatherLists];            // position of a list's first entry
  uint32_t n[kGatherLists];
  uint32_t first_block[kGatherLists];      // blocks of an eighth of all lists before it
  int32_t n_lists;
};
__global__ void __launch_bounds__(256)
stats_gather_lists_kernel(const int32_t* __restrict__ idx, const float* __restrict__ grad,
                          const float* __restrict__ hess, GatherTable t, uint32_t wrap, float* __restrict__ g_out,
                          float* __restrict__ h_out) {
  const uint32_t part = blockIdx.x % kXcds, b = blockIdx.x / kXcds;
  int32_t lo = 0, hi = t.n_lists - 1;  // the list that block b of this part is of (an empty list has no block)
  while (lo < hi) {
    const int32_t mid = (lo + hi + 1) >> 1;
    if (t.first_block[mid] <= b) {
      lo = mid;
    } else {
      hi = mid - 1;
    }
  }
  const uint32_t begin = t.first[lo], n = t.n[lo], each = (n + kXcds - 1) / kXcds;
  const uint32_t out = begin >= wrap ? begin - wrap : begin;
  const uint32_t at = part * each + (b - t.first_block[lo]) * (uint32_t)kGatherRows;
  const uint32_t part_end = (part + 1) * each < n ? (part + 1) * each : n;
  constexpr int kSteps = kGatherRows / 256;
  uint32_t row[kSteps];
#pragma unroll
  for (int i = 0; i < kSteps; ++i) {
    const uint32_t k = at + 256u * (uint32_t)i + threadIdx.x;
    row[i] = k < part_end ? (uint32_t)idx[begin + k] : 0u;
  }
  float g[kSteps], h[kSteps];
#pragma unroll
  for (int i = 0; i < kSteps; ++i) {
    const uint32_t k = at + 256u * (uint32_t)i + threadIdx.x;
    if (k < part_end) {
      g[i] = grad[row[i]];
      h[i] = hess[row[i]];
    }
  }
#pragma unroll
  for (int i = 0; i < kSteps; ++i) {
    const uint32_t k = at + 256u * (uint32_t)i + threadIdx.x;
    if (k < part_end) {
      g_out[out + k] = g[i];
      h_out[out + k] = h[i];
    }
  }
}

// Gradient and hessian of every row side by side, for a tree's builds: a leaf's scattered rows then
// fetch one line for both instead of two (see kStatsPairMinRows).
__global__ void __launch_bounds__(256)
stats_pair_kernel(const float* __restrict__ grad, const float* __restrict__ hess, int64_t n, float2* __restrict__ out) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
    out[i] = make_float2(grad[i], hess[i]);
}

// The unit counters of all tiles live at the head of the scratch workspace and are zero
// between calls: a workgroup's take is (workgroups per tile) + (old counter value), and
// the reduction pass, which follows every build that used them, sets them back to zero.
// This kernel zeroes them when a workspace is new.  (A fill kernel, not a memset node, so
// the call can be captured into a graph.)
__global__ void __launch_bounds__(256) counters_zero_kernel(uint32_t* counters, int32_t n_counters) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_counters) counters[i] = 0u;
}

// Several leaves in one launch.  Small leaves cannot fill the machine on their own (the
// synthetic benchmark of App. C.2 shows the rate falling with the leaf size); a level of
// a tree, or both children of a split, can.  The launch carries a table of up to
// kBatchLeaves leaves as kernel arguments -- nothing is staged through memory.  Leaf l
// (batch_plan.h) owns the row list idx[row_off .. row_off + n) and wgs workgroups per tile, which take
// its units of unit_epochs epochs in a fixed stride (no counters): a workgroup of leaf l
// runs build_tile exactly as a single-leaf launch in its fixed-split mode would, and the
// leaves' partial blocks lie back to back, each leaf's in the single-leaf order.  A leaf
// with one workgroup per tile writes its histogram itself and skips the reduction pass.
struct BatchArgs {
  const uint8_t* packed;
  const int32_t* idx;
  const float* grad;
  const float* hess;
  int32_t stats_by_pos;
  int32_t stat_shift;  // log2 of the bytes from a row's gradient to the next row's: 2, or 3 for (gradient, hessian) pairs
  uint32_t* partials;
  int64_t n_rows;
  int32_t n_main;
  int32_t wr;
  int32_t line_tiles;
  int32_t deal;
  int32_t n_leaves;
  uint32_t n_cols;       // workgroup columns of all leaves
  uint32_t stat_wrap;    // stats_by_pos: a list at idx position i has its statistics at i, or at i - this from this on
  gbdt_bin_t* hist_out;  // [n_leaves][n_features][n_bins]: written directly by leaves of one workgroup per tile
  int32_t n_features;
  int32_t n_bins;
  BatchLeaf leaf[kBatchLeaves];
};

// Words of the partial blocks one workgroup column (one workgroup of every tile) writes.
template <int CAP, int WM, bool NIB, int NT>
__device__ __host__ inline size_t column_words(int32_t n_main, int32_t wr) {
  size_t w = (size_t)n_main * block_words<CAP, WM, NIB, NT>();
  if (wr == 16) w += block_words<CAP, 16, NIB, NT>();
  if (wr == 32) w += block_words<CAP, 32, NIB, NT>();
  return w;
}

template <int CAP, int WM, bool NIB, int NT, int WPE, typename ACC, bool WIDE, bool HALVES, bool SHORT>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(WPE, WPE)))
hist_build_batch_kernel(BatchArgs a) {
  using BS = BuildShape<CAP, WM, NIB, NT, WIDE, HALVES>;
  __shared__ __align__(16) unsigned long long lds[BS::kLdsWords];
  const BatchBlock blk = BS::kHalves
                             ? batch_half_block(a.leaf, a.n_leaves, WM, a.n_main, a.deal, a.n_cols, blockIdx.x)
                             : batch_block(a.leaf, a.n_leaves, WM, a.n_main, a.wr, a.deal, a.n_cols, blockIdx.x);
  const BatchLeaf lf = a.leaf[blk.leaf];
  const int32_t wgs = (int32_t)batch_wgs(lf);
  const uint32_t unit_epochs = batch_unit_epochs(lf);
  constexpr int kPerWg = WIDE ? 2 : 1;  // partial blocks per workgroup
  const bool by_pos = a.stats_by_pos != 0;  // then grad / hess follow the row lists
  const uint32_t stat_off = !by_pos ? 0u : lf.row_off >= a.stat_wrap ? lf.row_off - a.stat_wrap : lf.row_off;
  uint32_t* leaf_out =
      a.partials + (size_t)lf.first_wg * kPerWg * column_words<CAP, WM, NIB, NT>(a.n_main, a.wr);
  build_part<CAP, WM, NIB, NT, ACC, true, WIDE, HALVES, SHORT>(
      a.packed, a.n_rows, a.n_main, a.wr, a.line_tiles, blk.tile, blk.half, leaf_out, (size_t)(kPerWg * wgs),
      (size_t)blk.wg, (size_t)wgs,
      wgs == 1 ? a.hist_out + (size_t)batch_leaf_no(lf) * a.n_features * a.n_bins : nullptr, a.n_features, a.n_bins, lds,
      a.idx + lf.row_off, a.grad + stat_off, a.hess + stat_off, by_pos,
      (uint32_t)a.stat_shift, lf.n, (uint32_t)blk.wg, 0u, unit_epochs, (uint32_t)wgs, (uint32_t*)nullptr, 0u, 0u);
}

}  // namespace

#endif  // GBDT_HIST_BUILD_KERNELS_H_
