// libgbdt_hist: feature-histogram construction, sibling subtraction, best-split scan,
// row partition and leaf-wise tree growth for histogram-based GBDT training on AMD
// gfx950 (MI355X).  This file holds the host side (launch planning, scratch, the C ABI);
// the kernels are in hist_build_kernels.h, hist_reduce_kernels.h, split_kernels.h and
// partition_kernels.h, the layouts in tile_plan.h and batch_plan.h.
// Method: arXiv 1706.08359 -- Alg. 1 (Sec. 3.3) defines the histogram, Sec. 4 /
// Alg. 2 / App. A.1 describe a GPU organisation for older hardware.  What is
// kept from that design: one lane handles a bundle of adjacent features of one
// sample (there 4 bytes, here up to 16); lanes that work in the same step are
// steered to different histogram columns by rotating the feature order per lane;
// work is split by features and by samples with a final reduction pass; small
// bin counts get cheaper variants.
// What is new here is stated at each kernel.
//
// Written for gfx950 only: 64-wide wavefronts, 160 KB LDS per CU, fast integer LDS
// atomics (ds_add_u64 / ds_add_u32; the float form ds_add_f32 is ~35x slower),
// 256 CUs in 8 XCDs.
#include <hip/hip_runtime.h>

#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <initializer_list>
#include <mutex>
#include <type_traits>
#include <unordered_map>
#include <utility>
#include <vector>

#include "../../include/gbdt_hist.h"
#include "tile_plan.h"
#include "batch_plan.h"

#include "hist_build_kernels.h"
#include "hist_reduce_kernels.h"
#include "split_kernels.h"
#include "partition_kernels.h"

// Scratch of the no-allocation entry point (gbdt_hist_build_noalloc): the unit counters
// (256 KiB head, as in every scratch buffer of this library) and up to 64 MiB of partial
// histograms.  One copy per GPU the library runs on, held until the process ends.  In host
// code this name is only a stand-in for the symbol: the device address is looked up once
// per device (noalloc_scratch_ptr) and that pointer is what kernels and fills receive.
constexpr size_t kNoAllocPartialBytes = (size_t)64 << 20;
constexpr size_t kNoAllocScratchBytes = (size_t)65536 * sizeof(uint32_t) + kNoAllocPartialBytes;
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

namespace {

// ------------------------------------------------------- calibration copy kernel

// Plain copy of n 16-byte words: a kernel of known HBM traffic (n * 16 bytes read, n *
// 16 bytes written) against which the memory counters of a profiler run are scaled.
__global__ void __launch_bounds__(256)
calibration_copy_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, size_t n) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = src[i];
}

// ------------------------------------------------------------------- host state

thread_local char g_hip_err[256] = "";

int hip_fail(hipError_t e, const char* what) {
  snprintf(g_hip_err, sizeof g_hip_err, "%s: %s", what, hipGetErrorString(e));
  return GBDT_EHIP;
}

#define HIP_TRY(expr)                                  \
  do {                                                 \
    hipError_t e_ = (expr);                            \
    if (e_ != hipSuccess) return hip_fail(e_, #expr);  \
  } while (0)

std::atomic<int> g_deterministic{0};
std::atomic<int> g_wide{0};  // wide (fp64-grade) accumulation, see gbdt_set_wide_accumulation

struct Workspace {
  std::mutex mu;
  void* own = nullptr;  // library-owned scratch
  size_t own_bytes = 0;
  int own_device = -1;
  std::vector<void*> retired;  // outgrown library buffers: work enqueued earlier may still use them
  void* user = nullptr;  // caller-registered scratch
  size_t user_bytes = 0;
  void* zeroed = nullptr;  // the buffer whose counter head is known to be all zero
};
Workspace g_ws;

// The head of every scratch buffer holds the build kernels' unit counters (one per
// feature tile, at most 65535 tiles); the scratch handed to a call starts behind it.
constexpr int kCounterSlots = 65536;
constexpr size_t kWsHeadBytes = (size_t)kCounterSlots * sizeof(uint32_t);
static_assert(kNoAllocScratchBytes == kWsHeadBytes + kNoAllocPartialBytes, "head of the fixed scratch");

bool stream_is_capturing(hipStream_t s) {
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &cs) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return cs == hipStreamCaptureStatusActive;
}

// Returns a scratch pointer of at least `bytes` for work enqueued on stream s, growing
// the library-owned buffer when no caller buffer is registered.  Growing allocates a
// new buffer and RETIRES the old one (kernels enqueued earlier may still use it; retired
// buffers are freed by gbdt_reset): no synchronisation, no free inside an enqueuing
// call.  It is refused (GBDT_ENOMEM) while s is being captured into a graph, where an
// allocation is not allowed: run the same call once outside the capture first, or
// register a caller buffer.  counters_out: the counter head of the same buffer;
// *counters_zero_out: whether it is known to be all zero.
int get_workspace(size_t bytes, hipStream_t s, void** out, uint32_t** counters_out = nullptr,
                  bool* counters_zero_out = nullptr) {
  std::lock_guard<std::mutex> lk(g_ws.mu);
  bytes += kWsHeadBytes;
  void* base = nullptr;
  if (g_ws.user) {
    if (bytes > g_ws.user_bytes) {
      snprintf(g_hip_err, sizeof g_hip_err, "caller workspace of %zu bytes, %zu needed", g_ws.user_bytes, bytes);
      return GBDT_ENOMEM;
    }
    base = g_ws.user;
  } else {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (!g_ws.own || g_ws.own_device != dev || g_ws.own_bytes < bytes) {
      if (stream_is_capturing(s)) {
        snprintf(g_hip_err, sizeof g_hip_err,
                 "library scratch must grow to %zu bytes, which is not possible during stream capture", bytes);
        return GBDT_ENOMEM;
      }
      size_t want = bytes < (size_t)(1 << 20) ? (size_t)(1 << 20) : bytes;
      if (g_ws.own && g_ws.own_device == dev && want < 2 * g_ws.own_bytes) want = 2 * g_ws.own_bytes;
      void* fresh = nullptr;
      hipError_t e = hipMalloc(&fresh, want);
      if (e != hipSuccess && want > bytes) e = hipMalloc(&fresh, want = bytes);
      if (e != hipSuccess) {
        hip_fail(e, "hipMalloc(workspace)");
        return GBDT_ENOMEM;
      }
      if (g_ws.own) g_ws.retired.push_back(g_ws.own);
      g_ws.own = fresh;
      g_ws.own_bytes = want;
      g_ws.own_device = dev;
    }
    base = g_ws.own;
  }
  *out = (char*)base + kWsHeadBytes;
  if (counters_out) *counters_out = (uint32_t*)base;
  if (counters_zero_out) *counters_zero_out = g_ws.zeroed == base;
  return GBDT_OK;
}

// Records whether the counter head of the buffer `counters` heads is all zero.
void set_counters_zero(uint32_t* counters, bool zero) {
  std::lock_guard<std::mutex> lk(g_ws.mu);
  if (zero) {
    g_ws.zeroed = counters;
  } else if (g_ws.zeroed == counters) {
    g_ws.zeroed = nullptr;
  }
}

// Device address of `scratch` on the current device, looked up on the first call there
// (every GPU holds its own copy of the array at its own address).
constexpr int kMaxDevices = 64;
int noalloc_scratch_ptr(void** out) {
  static std::mutex mu;
  static void* ptr[kMaxDevices] = {};
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return GBDT_EUNSUPPORTED;
  std::lock_guard<std::mutex> lk(mu);
  if (!ptr[dev]) {
    void* q = nullptr;
    HIP_TRY(hipGetSymbolAddress(&q, HIP_SYMBOL(scratch)));
    if (!q) return GBDT_EHIP;
    ptr[dev] = q;
  }
  *out = ptr[dev];
  return GBDT_OK;
}

// ---- fused columns (see FusedCol in hist_build_kernels.h): which packed matrices have a fused
// copy, keyed by the address gbdt_bins_pack wrote them to
struct FusedEntry {
  const uint8_t* tiles = nullptr;     // the fused copy's feature tiles
  const FusedFeat* feats = nullptr;   // [n_features] on the device, inside the fused copy
  int64_t n_rows = 0;
  int32_t n_features = 0, n_bins = 0, n_cols = 0;
};
std::mutex g_fused_mu;
std::unordered_map<const void*, FusedEntry> g_fused;

bool fused_lookup(const void* packed, int64_t n_rows, int32_t n_features, int32_t n_bins, FusedEntry* out) {
  static const bool off = [] {
    const char* e = getenv("GBDT_HIST_NO_FUSE");  // tuning experiments: always build from the plain tiles
    return e && atoi(e) > 0;
  }();
  if (off) return false;
  std::lock_guard<std::mutex> lk(g_fused_mu);
  auto it = g_fused.find(packed);
  if (it == g_fused.end()) return false;
  const FusedEntry& e = it->second;
  if (e.n_rows != n_rows || e.n_features != n_features || e.n_bins != n_bins) return false;
  *out = e;
  return true;
}

// Leaves below this many rows are built from the plain tiles: the extra launch that takes the
// marginals costs more than the atomics the fused columns save.
constexpr int64_t kFusedMinLeafRows = 8192;
// ... and leaves that hold less than a third of the matrix's rows: a gathered row drags its whole
// 128-byte line along, so sparse leaves are bound by HBM traffic, and a fused copy's rows are wider
// than 4-bit rows (measured on 11 M x 700 with 2..16 levels: 0.78x the time at half of the rows and
// more, break-even at a quarter, 1-3 % slower below).
constexpr int64_t kFusedMinLeafFraction = 3;
// A fused copy is made when it has at most this fraction of the features as columns.
constexpr double kFusedMaxColumnRatio = 0.85;
constexpr int64_t kFuseSampleRows = 4096;  // rows gbdt_bins_fuse looks at before it reads them all ...
constexpr int64_t kFuseSampleMinRows = 65536;  // ... of a matrix of so many rows ...
constexpr int64_t kFuseSampleMinBytes = (int64_t)1 << 25;  // ... and bytes
// (A look is a launch and a round trip to the host more, 24 us where it proves nothing; where it does, the
// second launch is saved, and the reading.  Looking first from 65,536 rows on, whatever the bytes: 66,000 x 8 x 16, not
// fused, 48 -> 61 us, and 36 without the look; 1,000,000 x 10 x 16 65 and 40 us.  Provably full: 800,000 x 40 x 64
// 34 us with and 41 without, 2,000,000 x 40 x 64 34 and about 60.)
int64_t fuse_sample_rows(int64_t n_rows, int32_t n_features) {
  return n_rows >= kFuseSampleMinRows && n_rows * n_features >= kFuseSampleMinBytes ? kFuseSampleRows : 0;
}

// Packs features into columns of at most kFusedCap joint levels: features in descending order
// of their level counts, each into the fullest column that still takes it (best fit).
void plan_fusion(const std::vector<uint32_t>& levels, std::vector<FusedCol>* cols, std::vector<FusedFeat>* feats) {
  const int32_t F = (int32_t)levels.size();
  std::vector<int32_t> order(F);
  for (int32_t f = 0; f < F; ++f) order[f] = f;
  std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return levels[a] > levels[b]; });
  std::vector<uint32_t> prod;                          // joint levels of every column so far
  std::vector<std::vector<int32_t>> open(kFusedCap + 1);  // columns by joint levels, with room for another part
  cols->clear();
  feats->assign(F, FusedFeat{});
  for (int32_t f : order) {
    const uint32_t L = levels[f] < 1 ? 1 : levels[f];
    int32_t c = -1;
    for (uint32_t pr = kFusedCap / L; pr >= 1 && c < 0; --pr) {
      if (!open[pr].empty()) {
        c = open[pr].back();
        open[pr].pop_back();
      }
    }
    if (c < 0) {
      c = (int32_t)cols->size();
      FusedCol col;
      for (int k = 0; k < kFusedMaxParts; ++k) {
        col.feature[k] = -1;
        col.stride[k] = 0;
      }
      col.n_parts = 0;
      col.pad = 0;
      cols->push_back(col);
      prod.push_back(1);
    }
    FusedCol& col = (*cols)[c];
    col.feature[col.n_parts] = f;
    col.stride[col.n_parts] = (uint8_t)prod[c];
    FusedFeat& ff = (*feats)[f];
    ff.col = c;
    ff.stride = (uint8_t)prod[c];
    ff.levels = (uint8_t)L;
    ff.pad[0] = ff.pad[1] = 0;
    col.n_parts += 1;
    prod[c] *= L;
    if (col.n_parts < kFusedMaxParts && prod[c] <= kFusedCap) open[prod[c]].push_back(c);
  }
}

// Byte layout of a fused copy with n_cols columns: [feature tiles][slack][FusedFeat x n_features][FusedCol x n_cols]
struct FusedLayout {
  TilePlan plan;
  size_t feats_off, cols_off, total;
};
FusedLayout fused_layout(int64_t n_rows, int32_t n_features, int32_t n_cols) {
  FusedLayout l;
  l.plan = make_tile_plan(n_cols, kFusedCap);
  const size_t tiles = (size_t)n_rows * l.plan.row_bytes + (size_t)kPlanSlackBytes;
  l.feats_off = (tiles + 255) / 256 * 256;
  l.cols_off = (l.feats_off + (size_t)n_features * sizeof(FusedFeat) + 255) / 256 * 256;
  l.total = (l.cols_off + (size_t)n_cols * sizeof(FusedCol) + 255) / 256 * 256;
  return l;
}

// Optional timing of the build kernel alone (it shares its C-ABI call with the merge
// kernel): when enabled, every gbdt_hist_build records a HIP event on the call's
// stream right before and right after the build kernel.
struct Profile {
  std::mutex mu;
  bool on = false;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> pairs;
};
Profile g_prof;

int device_cu_count() {
  static int cached_dev = -1, cached_cus = 0;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  if (dev != cached_dev) {
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
      cus = 256;
    cached_cus = cus;
    cached_dev = dev;
  }
  return cached_cus;
}

constexpr size_t kLdsPerCu = 160 * 1024;
constexpr int64_t kPackStreamBytes = (int64_t)256 << 20;  // the memory-side cache; see pack_kernel
static_assert(kPlanSlackBytes == (int64_t)kEpochRows * 64, "slack behind the tiles: one epoch of the widest tile");
constexpr int kBuildThreads = 512;  // threads per workgroup of every build kernel variant

struct BuildGeom {
  TilePlan plan;
  int nt;               // threads per workgroup
  size_t lds_bytes;     // LDS per workgroup
  int wgs;              // workgroups per tile
  int unit_epochs;      // epochs per unit
  bool one_unit_each;   // short leaf: every workgroup has exactly one unit, no counter
  int blocks_per_wg;    // partial blocks a workgroup writes: 1, or 2 with wide accumulation
  bool halves;          // main tiles are built in halves (plan_halves)
  int parts;            // tiles, or halves and the remainder tile
  size_t partial_words;  // total words of all partial blocks
};

// Leaves of at most this many epochs get ONE workgroup per tile, which writes the
// finished histogram itself: a second launch (the reduction pass) would cost more than
// the few epochs a second workgroup could take over.
constexpr int kDirectEpochs = 4;

// When an index-list build gathers grad / hess into leaf order first: with several feature
// tiles (each would gather the same scattered values again), a leaf that is sparse in the
// matrix (scattered 4-byte reads cost a memory sector each) and big enough for the saving
// to exceed one more small launch.  While the two arrays fit an XCD's L2 (4 MB) the tiles'
// gathers mostly hit there and only leaves below a fifth of the rows gain; beyond that,
// leaves up to half of the rows do.  Measured: 10-45 % off the build kernel of such leaves
// on the 137-, 500- and 700-feature matrices.
constexpr int kStatsGatherMinTiles = 4;
constexpr int64_t kStatsGatherMinRows = 8192;
bool stats_gather_pays(int n_tiles, int64_t list_rows, int64_t rows_per_leaf, int64_t n_rows) {
  const int64_t dense_limit = n_rows >= (1 << 20) ? 2 : 5;  // leaf holds at most 1/2 or 1/5 of the rows
  return n_tiles >= kStatsGatherMinTiles && list_rows >= kStatsGatherMinRows &&
         rows_per_leaf * dense_limit <= n_rows;
}

// From this many rows on grad and hess do not fit an XCD's L2, and several lists are gathered by parts of the rows.  (Eight
// leaves of 200,000 x 100 x 255, build and partition: 41.8 us in list order, 43.2 by parts.)
constexpr int64_t kGatherListsMinRows = 1 << 19;

// Batches of matrices of two and three tiles that are built in halves (plan_halves): four and more parts, each of which would
// gather the scattered values, so small leaves of a matrix whose arrays do not fit an XCD's L2 are gathered first as well.
// (4,000,000 rows with wide sums, 64 leaves of all rows: 64 features 298 us by row id, 243 gathered, 96 features 518 and 388; 32
// leaves of half of the rows 157 and 140, 286 and 220.  Four leaves of half of the rows: 118 and 125, 168 and 169.  64 leaves of 1,000,000 x
// 64: 81 and 81.)
bool stats_gather_of_parts_pays(int n_parts, int64_t list_rows, int64_t rows_per_leaf, int64_t n_rows) {
  return n_parts >= kStatsGatherMinTiles && list_rows >= kStatsGatherMinRows && n_rows >= (1 << 20) &&
         rows_per_leaf * 32 <= n_rows;
}

// When a tree's leaves are not gathered that way (few tiles), gbdt_grow_tree lays gradient and hessian
// of every row side by side once: a scattered row then costs one line of statistics instead of two, beside
// its line of bins.  From the size on at which both arrays no longer fit an XCD's L2.
// (255 leaves of 10.5 M x 28 x 255 bins: the tree's batched builds 1,570 -> 1,350 us, laying out the pairs 26.)
constexpr int64_t kStatsPairMinRows = 1 << 20;
bool stats_pair_pays(int n_tiles, int64_t n_rows) {
  return n_tiles < kStatsGatherMinTiles && n_rows >= kStatsPairMinRows && n_rows < ((int64_t)1 << 29);  // (32-bit offsets)
}

// Workgroups per tile and epochs per unit for a leaf of n_epochs epochs that may use
// `budget` workgroups per tile: units of kUnitEpochs handed out at run time when every
// workgroup gets more than kEvenSplitUnits of them; otherwise (short leaf) the epochs are
// split evenly, one unit per workgroup, and the unit counter is not needed
// (*one_unit_each_out).  With only a few units each, what the run-time hand-out gains in
// balance is less than what whole units lose: a workgroup with 2 units of 4 epochs waits
// for one with 3, while 10 or 11 epochs each end together (measured: 4-19 % on leaves of
// 10-25 % of the rows, nothing lost elsewhere).
constexpr int kEvenSplitUnits = 3;
void plan_leaf_units(int64_t n_epochs, int64_t budget, int* wgs_out, int* unit_epochs_out,
                     bool* one_unit_each_out) {
  int64_t wgs = budget;
  if (wgs > n_epochs) wgs = n_epochs;
  if (n_epochs <= kDirectEpochs) wgs = 1;
  if (wgs < 1) wgs = 1;
  int unit_epochs = kUnitEpochs;
  bool one_each = false;
  if (wgs * kUnitEpochs * kEvenSplitUnits >= n_epochs) {
    unit_epochs = (int)((n_epochs + wgs - 1) / wgs);
    if (unit_epochs < 1) unit_epochs = 1;
    const int64_t n_units = (n_epochs + unit_epochs - 1) / unit_epochs;
    if (n_units >= 1 && wgs > n_units) wgs = n_units;  // no workgroup without a unit
    one_each = true;
  }
  *wgs_out = (int)wgs;
  *unit_epochs_out = unit_epochs;
  *one_unit_each_out = one_each;
}

// A leaf of more units than that: every workgroup starts with one long unit, which together hold this
// share of the epochs, and only the rest is handed out at run time, in small units, to even out
// the ends.  A workgroup then reads one stretch of rows for most of its life instead of a piece here and a
// piece there, and workgroups that share cache lines stay side by side.  Measured against units of 4
// epochs handed out from the start: categorical root (fused columns) 289 -> 258 us, dense_wide root with a
// region per tile 176 -> 170 us, dense_tall root 129 -> 124 us; 85 to 98 % are within 2 % of each other, and
// tiles that share lines want the most (dense_wide root 181 us at 85 %, 179 at 95).
// Not so a list whose tiles share no lines (a lone tile, fused columns, the largest matrices): hundreds of
// stretches of scattered rows at once are a little slower than one front of small units that goes through the list.
// 40,000,000 x 60 x 64, a list of half the rows: 439 us with long first units, 415 with units of 4 epochs (and 498 /
// 466 on a first pass); the fused columns of 3,000,000 x 700 x 16, half of the rows: 222 / 214 and 269 / 256.
// 4-bit tiles with a narrower last one: of the four workgroups of a CU one may be of the narrow tile, done in half
// the time, and those beside it then run ahead, so more is left to even out (11,000,000 x 700 x 16, root 1,500 us at 95 %,
// 1,444 at 85, 1,410 at 75 and at 60, 1,411 with units of 4 from the start).
constexpr int kFirstUnitPercent = 95;
constexpr int kFirstUnitPercentUneven = 75;
constexpr int kTailUnitEpochs = 3;  // the fewest the pipeline's look-ahead allows
static_assert(kTailUnitEpochs >= 3, "a unit's successor is taken in its third-last epoch");

// Chooses the grid: as many workgroups per tile as fit the machine at once (they stay
// until their tile's units are used up), and the unit size.  wg_per_cu: resident
// workgroups per CU of the kernel variant as reported by the runtime (<= 0: estimate
// from the LDS footprint alone).
BuildGeom make_geom(int32_t n_features, int32_t n_bins, int64_t n_leaf, int cus,
                    int wg_per_cu_hint, bool wide = false, bool halves = false, int64_t max_wgs = (int64_t)1 << 40) {
  BuildGeom g;
  g.plan = make_tile_plan(n_features, n_bins);
  g.halves = halves;
  g.parts = plan_n_parts(g.plan, halves);
  const TilePlan& p = g.plan;
  g.nt = kBuildThreads;
  g.blocks_per_wg = wide ? 2 : 1;
  const size_t main_block = (size_t)3 * plan_cells(p, p.wm);  // (of both halves where tiles are built so)
  const size_t wg_cells = plan_cells(p, halves ? 16 : p.wm);
  g.lds_bytes = wg_cells * 8 * g.blocks_per_wg + 4 * (g.nt / 64) * sizeof(float) + 8;
  int wg_per_cu = wg_per_cu_hint;
  if (wg_per_cu <= 0) {
    wg_per_cu = (int)(kLdsPerCu / g.lds_bytes);
    const int by_threads = 2048 / g.nt;
    if (wg_per_cu > by_threads) wg_per_cu = by_threads;
  }
  if (wg_per_cu < 1) wg_per_cu = 1;
  const int64_t resident = (int64_t)cus * wg_per_cu;
  const int64_t n_epochs = (n_leaf + kEpochRows - 1) / kEpochRows;
  // (A narrow tile's epochs are cheaper, but not by much: the per-epoch overhead does
  // not shrink with the tile.  It gets as many workgroups as a main tile.)
  int64_t budget = resident / g.parts;
  if (budget > max_wgs) budget = max_wgs;
  plan_leaf_units(n_epochs, budget, &g.wgs, &g.unit_epochs, &g.one_unit_each);
  // (a 16-byte tile of 256 bins needs half of what is set aside for it)
  g.partial_words = ((size_t)p.n_main * g.wgs * main_block +
                     (size_t)(p.wr ? g.wgs : 0) * 3 * (p.wr ? (size_t)plan_pages(p, p.wr) * p.cap * 32 : 0)) *
                    g.blocks_per_wg;
  return g;
}

// How the workgroups of a tile share out a leaf's epochs, and how the launch's blocks are dealt out.
struct UnitPlan {
  int32_t unit_epochs;
  int32_t first_epochs;  // 0, or the length of every workgroup's first unit
  int32_t fixed_stride;  // 0: units from the tile's counter
  int32_t deal;          // order of the launch's blocks (batch_plan.h)
};
UnitPlan plan_units(const BuildGeom& g, int64_t n_leaf, bool indexed, int32_t line_tiles, bool deterministic, int cus) {
  UnitPlan u;
  u.unit_epochs = g.unit_epochs;
  u.first_epochs = 0;
  if (!g.one_unit_each) {
    const int64_t n_epochs = (n_leaf + kEpochRows - 1) / kEpochRows;
    if (deterministic) {  // an even split: the same sums in every run, and rows stay together
      u.unit_epochs = (int32_t)((n_epochs + g.wgs - 1) / g.wgs);
    } else {
      const int percent = g.plan.nib && g.plan.wr ? kFirstUnitPercentUneven : kFirstUnitPercent;
      const int32_t first = (int32_t)(n_epochs * percent / 100 / g.wgs);
      const bool lines = (line_tiles > 1 && g.plan.n_main > 1) || g.halves;
      if (first >= kUnitEpochs && (!indexed || lines)) {
        u.first_epochs = first;
        u.unit_epochs = kTailUnitEpochs;
      }
    }
  }
  // no counter when every workgroup has one unit anyway, or when the split must be fixed
  // (... or when there are more parts than counters)
  u.fixed_stride = (g.one_unit_each || deterministic || g.parts > kCounterSlots) ? g.wgs : 0;
  u.deal = deal_order(line_tiles, g.unit_epochs, (int64_t)g.wgs * g.parts, cus, g.blocks_per_wg > 1);
  return u;
}

// Which of its two kernels a leaf takes.  SHORT spends less on the leaf's end: its last epoch, and the histogram, which a tile's only
// workgroup writes.  The other one spends less on every epoch, and its last one may as well add zeros beside workgroups that are full.
// SHORT and long us: one workgroup a tile, 28 x 255, an epoch 6.2 and 7.0, four 11.7 and 12.6; 60 x 64 5.9 and 6.5, 12.4 and 13.0; 400 x 16,
// wide, 9.3 and 10.2, 28.2 and 28.7.  Several, 256 bins, of one epoch, root of 100,000 x 28 19.0 and 21.5, of two, 32,700 of 500 features 27.8
// and 29.1, of three 29.0 and 28.9, of ten, a tenth of 1,500,000 x 500 as a list 49.7 and 49.0.  64 bins, of one to twelve epochs, 0 to 1 % more
// SHORT (a fiftieth of 8,000,000 x 500 as a list 43.3 and 42.8); 16 bins, a tenth of 3,000,000 x 400 as a list 47.4 and 46.3.
constexpr int kShortUnitEpochs = 2;
bool leaf_is_short(const BuildGeom& g, bool wide) {
  if (wide && g.plan.cap == 256) return true;  // (one kernel for both)
  return g.one_unit_each && (g.wgs == 1 || (g.plan.cap == 256 && g.unit_epochs <= kShortUnitEpochs));
}

// How the rows of a build lie in the matrix, for plan_halves.  Sparse: a list of at most a fifth of the rows, and all leaves of
// a batch.  Many sparse rows: from kSparseManyRows listed ones on, in a batch if its leaves hold at most a twelfth of the rows
// each on average (1,000,000 x 33 x 255: 32 leaves of half of the rows 45.9 us whole, 54.7 in halves, 64 of all 76 and 79;
// 300,000 x 33 x 255: 64 of all 41 and 30; 4,000,000 x 33 x 255: four leaves of half of the rows 119 and 95), half as many in one
// list (2,000,000 x 33 x 255, a tenth 27.6 and 29.7, 1,000,000, 19 % 26.4 and 25.5).
// Large: many sparse rows of a matrix of kLargeMatrixRows on (64 features, 64 leaves of all rows: 4,000,000 252 us whole, 243 in
// halves, 10,000,000 580 and 639; 96 features, a tenth in one list: 7,000,000 74.2 and 76.7, 4,000,000 50.7 and 47.1).
constexpr int64_t kSparseManyRows = 384 * 1024;
constexpr int64_t kLargeMatrixRows = 1 << 23;
int rows_of_leaf(bool indexed, int64_t n_leaf, int64_t n_rows) {
  if (!indexed || n_leaf > n_rows / 5) return kRowsDense;
  if (n_leaf < kSparseManyRows / 2) return kRowsSparse;
  return n_rows >= kLargeMatrixRows ? kRowsLargeList : kRowsSparseMany;
}
int rows_of_batch(int64_t total_rows, int32_t n_leaves, int64_t n_rows) {
  if (total_rows < kSparseManyRows || total_rows / n_leaves * 12 > n_rows) return kRowsSparse;
  return n_rows >= kLargeMatrixRows ? kRowsLargeBatch : kRowsSparseMany;
}

// Kernel variants: bin capacity -> (main tile width, 4-bit, waves per SIMD the
// register budget is set for).
#define GBDT_VARIANT_16 16, 64, true, kBuildThreads, 8, double
#define GBDT_VARIANT_64 64, 64, false, kBuildThreads, 6, float
#define GBDT_VARIANT_256 256, 32, false, kBuildThreads, 4, float
// The same with wide accumulation: twice the LDS, fp64 accumulators.
#define GBDT_VARIANT_16W 16, 64, true, kBuildThreads, 6, double
#define GBDT_VARIANT_64W 64, 64, false, kBuildThreads, 4, double
#define GBDT_VARIANT_256W 256, 32, false, kBuildThreads, 2, double
#define GBDT_VARIANT_256W_HALVES 256, 32, false, kBuildThreads, 4, double

template <int CAP, int WM, bool NIB, int NT, int WPE, typename ACC, bool INDEXED, bool WIDE = false, bool HALVES = false>
int query_occupancy() {
  int n = 0;
  hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
      &n, reinterpret_cast<const void*>(hist_build_kernel<CAP, WM, NIB, NT, WPE, ACC, INDEXED, WIDE, HALVES, WIDE && CAP == 256>),
      NT, 0);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  return n;
}

// Resident workgroups per CU of the build kernel variant for this bin capacity
// (registers, LDS and wave slots taken into account by the runtime); cached.
int build_wg_per_cu(int cap, bool indexed, bool wide = false, bool halves = false) {
  // GBDT_HIST_WG_PER_CU overrides the runtime's answer (tuning experiments only)
  if (const char* e = getenv("GBDT_HIST_WG_PER_CU")) {
    const int v = atoi(e);
    if (v > 0) return v;
  }
  static int cache[7][2] = {{-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}};
  const int ci = cap == 16 ? 0 : (cap == 64 ? 1 : 2);
  int& c = cache[halves ? 6 : ci + (wide ? 3 : 0)][indexed ? 1 : 0];
  if (c < 0 && halves) {
    c = indexed ? query_occupancy<GBDT_VARIANT_256W_HALVES, true, true, true>()
                : query_occupancy<GBDT_VARIANT_256W_HALVES, false, true, true>();
  }
  if (c < 0 && wide) {
    if (cap == 16) c = indexed ? query_occupancy<GBDT_VARIANT_16W, true, true>() : query_occupancy<GBDT_VARIANT_16W, false, true>();
    else if (cap == 64) c = indexed ? query_occupancy<GBDT_VARIANT_64W, true, true>() : query_occupancy<GBDT_VARIANT_64W, false, true>();
    else c = query_occupancy<GBDT_VARIANT_256W, true, true>();  // (only lists are built so)
  }
  if (c < 0) {
    if (cap == 16) c = indexed ? query_occupancy<GBDT_VARIANT_16, true>() : query_occupancy<GBDT_VARIANT_16, false>();
    else if (cap == 64) c = indexed ? query_occupancy<GBDT_VARIANT_64, true>() : query_occupancy<GBDT_VARIANT_64, false>();
    else c = indexed ? query_occupancy<GBDT_VARIANT_256, true>() : query_occupancy<GBDT_VARIANT_256, false>();
  }
  return c;
}

// Work split of split_gain_kernel over the n_hists histograms of a launch.  group: features of a wavefront's
// step; passes: steps a workgroup takes; waves: its wavefronts; n_wg: workgroups, and candidates, per histogram.
// A wavefront takes one step while all of them fit the machine at once (four a SIMD: the kernel needs 122
// registers), then several.  Up to kSplitMaxWaves steps are one workgroup's, and nothing is handed
// over (28 x 64: 3.8 us, in two workgroups 4.9).  Beyond, workgroups are small -- 28 x 255 takes 5.4 us with four wavefronts
// each, 5.8 with 8 and 6.6 with 16 -- until the hand-off queues at the ticket: 2,000 x 63 6.5 us in 125 workgroups, 6.2 in
// 63; 2,000 x 255 12.7 in 500, 8.7 in 125.
constexpr int kSplitFitWaves = 4096;  // 256 CUs x 4 SIMDs x 4
constexpr int kSplitFewWgs = 64;
struct SplitGrouping {
  int group, passes, waves, n_wg;
};
SplitGrouping split_grouping(int32_t n_features, int32_t n_bins, int32_t n_hists) {
  SplitGrouping g;
  g.group = 64 >> split_lane_bits(n_bins);
  const int64_t n_steps = ((int64_t)n_features + g.group - 1) / g.group;
  int64_t each = (n_steps * (n_hists > 0 ? n_hists : 1) + kSplitFitWaves - 1) / kSplitFitWaves;  // steps of a wavefront
  if (n_steps <= kSplitMaxWaves) {
    if (each > 4) each = 4;
    g.waves = (int)((n_steps + each - 1) / each);
    g.passes = (int)n_steps;
    g.n_wg = 1;
    return g;
  }
  // never more workgroups than a lone histogram gets: the scratch is sized by that
  const int64_t most = n_hists > 1 ? split_grouping(n_features, n_bins, 1).n_wg : n_steps;
  g.waves = 4;
  if (each > (n_steps + g.waves - 1) / g.waves) each = (n_steps + g.waves - 1) / g.waves;
  for (;; g.waves *= 2) {
    g.passes = (int)(each * g.waves);
    g.n_wg = (int)((n_steps + g.passes - 1) / g.passes);
    if (g.waves >= kSplitMaxWaves || (g.n_wg <= kSplitFewWgs && g.n_wg <= most)) return g;
  }
}

// GBDT_HIST_CHECK_INPUTS=1 (debugging): every call that takes a row list first counts its
// out-of-range entries on the device, WAITS for the stream and fails with GBDT_EINVAL if
// there are any, instead of the undefined behaviour of the unchecked path.
bool check_inputs_enabled() {
  static const bool on = [] {
    const char* e = getenv("GBDT_HIST_CHECK_INPUTS");
    return e && atoi(e) > 0;
  }();
  return on;
}

int check_row_ids(const int32_t* idx, int64_t n, int64_t n_rows, hipStream_t s) {
  if (!check_inputs_enabled() || !idx || n <= 0) return GBDT_OK;
  void* ws = nullptr;
  int rc = get_workspace(256, s, &ws);
  if (rc != GBDT_OK) return rc;
  unsigned long long* n_bad = (unsigned long long*)ws;
  hipLaunchKernelGGL(counters_zero_kernel, dim3(1), dim3(256), 0, s, (uint32_t*)ws, 2);
  HIP_TRY(hipGetLastError());
  const int64_t blocks = (n + 255) / 256;
  hipLaunchKernelGGL(row_ids_check_kernel, dim3((unsigned)(blocks < 4096 ? blocks : 4096)), dim3(256), 0, s, idx,
                     n, n_rows, n_bad);
  HIP_TRY(hipGetLastError());
  unsigned long long bad = 0;
  HIP_TRY(hipMemcpyAsync(&bad, n_bad, sizeof bad, hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  if (bad) {
    snprintf(g_hip_err, sizeof g_hip_err, "%llu row ids outside [0, n_rows)", bad);
    return GBDT_EINVAL;
  }
  return GBDT_OK;
}

bool valid_shape(int64_t n_rows, int32_t n_features, int32_t n_bins) {
  return n_rows >= 0 && n_features > 0 && n_bins >= 2 && n_bins <= 256;
}

// Brackets the build kernel with events while profiling is enabled.
struct BuildTimer {
  hipEvent_t ev0 = nullptr, ev1 = nullptr;
  bool on = false;
  int begin(hipStream_t s) {
    {
      std::lock_guard<std::mutex> lk(g_prof.mu);
      on = g_prof.on;
    }
    if (on) {
      HIP_TRY(hipEventCreate(&ev0));
      HIP_TRY(hipEventCreate(&ev1));
      HIP_TRY(hipEventRecord(ev0, s));
    }
    return GBDT_OK;
  }
  int end(hipStream_t s) {
    if (on) {
      HIP_TRY(hipEventRecord(ev1, s));
      std::lock_guard<std::mutex> lk(g_prof.mu);
      g_prof.pairs.emplace_back(ev0, ev1);
    }
    return GBDT_OK;
  }
};

template <int CAP, int WM, bool NIB, int NT, int WPE, typename ACC, bool WIDE = false, bool HALVES = false, bool LISTS_ONLY = false>
int launch_build(const BuildArgs& a, int blocks, hipStream_t s, bool timed, bool is_short) {
  BuildTimer timer;
  int rc = timed ? timer.begin(s) : GBDT_OK;
  if (rc != GBDT_OK) return rc;
  auto launch = [&](auto short_tag) {
    constexpr bool kShort = decltype(short_tag)::value;
    if (a.idx) {
      hipLaunchKernelGGL((hist_build_kernel<CAP, WM, NIB, NT, WPE, ACC, true, WIDE, HALVES, kShort>), dim3(blocks), dim3(NT), 0,
                         s, a);
    } else if constexpr (!LISTS_ONLY) {
      hipLaunchKernelGGL((hist_build_kernel<CAP, WM, NIB, NT, WPE, ACC, false, WIDE, HALVES, kShort>), dim3(blocks), dim3(NT), 0,
                         s, a);
    }
  };
  if (is_short) {
    launch(std::true_type{});
  } else if constexpr (!(WIDE && CAP == 256)) {
    launch(std::false_type{});
  }
  HIP_TRY(hipGetLastError());
  return timer.end(s);
}

// Whether batches have a kernel for long leaves, beside SHORT (batch_is_short).
constexpr bool batch_has_long(int cap, bool wide) { return cap == 64 || (cap == 256 && !wide); }

template <int CAP, int WM, bool NIB, int NT, int WPE, typename ACC, bool WIDE = false, bool HALVES = false>
int launch_build_batch(const BatchArgs& a, int blocks, hipStream_t s, bool is_short) {
  BuildTimer timer;
  int rc = timer.begin(s);
  if (rc != GBDT_OK) return rc;
  if (is_short) {
    hipLaunchKernelGGL((hist_build_batch_kernel<CAP, WM, NIB, NT, WPE, ACC, WIDE, HALVES, true>), dim3(blocks), dim3(NT), 0, s, a);
  } else if constexpr (batch_has_long(CAP, WIDE)) {
    hipLaunchKernelGGL((hist_build_batch_kernel<CAP, WM, NIB, NT, WPE, ACC, WIDE, HALVES, false>), dim3(blocks), dim3(NT), 0, s, a);
  }
  HIP_TRY(hipGetLastError());
  return timer.end(s);
}

template <int CAP, int WM, bool NIB, int NT, int WPE, typename ACC>
size_t variant_column_words(const TilePlan& p) {
  return column_words<CAP, WM, NIB, NT>(p.n_main, p.wr);
}

// Plan of one batched launch: leaves [l0, l0 + n) of the call share the machine, at least one
// workgroup per tile each, so that the launch ends early: with T the most epochs a workgroup
// gets, leaf i takes ceil(epochs / T) workgroups per tile ("columns" of workgroups).  Either all columns
// fit the machine at once and the launch lasts T epochs, or columns are dealt out, the longest first, as places
// come free, and it lasts their average and half of a last one.  A column costs kBatchColumnEpochs on
// top (clearing and draining its histograms, filling its pipeline, writing its sums), a leaf of several
// columns the reduction pass over them: kBatchMergeEpochs of a column for every block of sums written or
// read.  T is the cheapest of a dozen candidates around the average of one machine-full of columns.  (Shares of the machine rounded
// down, as it was, left the largest of 64 leaves of 1.5 M x 500 x 255 bins alone with 167 epochs
// where the average place had 92: 787 us, now 440.)
struct BatchPlan {
  BatchLeaf leaf[kBatchLeaves];  // most epochs per workgroup first
  int n = 0;
  int n_live = 0;          // leaves with rows
  uint32_t total_wgs = 0;  // workgroups per tile over all leaves
  int most_unit_epochs = 1;
  uint32_t most_each = 0;  // epochs of the busiest workgroup
};
constexpr double kBatchColumnEpochs = 3.0;
constexpr double kBatchMergeEpochs = 2.0;
constexpr double kBatchMergeLaunchEpochs = 1.5;
// An epoch takes as long as the other workgroups of its CU let it: with k of the w that fit a CU at once it
// takes about 0.2 + 0.8 k / w of the time with all of them; the 256-bin variant, of which two fit and which is
// bound by vector work as much as by what they share, 0.4 + 0.6 k / w (5,050 cycles alone, 7,090 together).  A plan of
// fewer columns can so be as fast, and it has fewer sums to reduce and fewer rows of the matrix in flight.
// What counts is the fullest CU, so counts of workgroups just at or under a multiple of the CUs are tried too.
// (8,000,000 x 500 x 64, 64 equal leaves: one column each, two workgroups a CU, 1,290 us, two columns each, which a
// plan prefers that takes an epoch to last the same always, 1,650; 11,000,000 x 300 x 16, 64 equal leaves: four columns
// each, exactly three workgroups a CU, 810 us, five 1,270.)
constexpr double kBatchAloneShare = 0.2, kBatchAloneShareOfTwo = 0.4;
constexpr int kBatchMaxPerCu = 8;

BatchPlan plan_batch(const int64_t* leaf_offsets, int32_t l0, int32_t n, int cus, int wg_per_cu,
                     int n_tiles, const uint32_t* seg_off = nullptr) {
  const int64_t resident = (int64_t)cus * wg_per_cu;
  BatchPlan b;
  b.n = n;
  uint32_t epochs[kBatchLeaves], most = 1;  // (leaves hold fewer than 2^31 rows)
  uint32_t longer[kBatchLeaves];  // the leaves whose columns depend on T: those of more than kDirectEpochs epochs
  int64_t total_epochs = 0;
  int n_long = 0;
  for (int i = 0; i < n; ++i) {
    epochs[i] = (uint32_t)((leaf_offsets[l0 + i + 1] - leaf_offsets[l0 + i] + kEpochRows - 1) / kEpochRows);
    total_epochs += epochs[i];
    if (epochs[i] > most) most = epochs[i];
    b.n_live += epochs[i] > 0;
    if (epochs[i] > (uint32_t)kDirectEpochs) longer[n_long++] = epochs[i];
  }
  int64_t budget = resident / n_tiles;
  if (budget < 1) budget = 1;
  uint32_t t = most;
  double t_cost = 1e300;
  double share[kBatchMaxPerCu] = {0};
  if (wg_per_cu > kBatchMaxPerCu) wg_per_cu = kBatchMaxPerCu;
  auto consider = [&](uint32_t cand) {
    // ceil(e / cand) by a multiplication: e and cand are below 2^22, so quotients that are no whole numbers are
    // at least 2^-22 away from one, and 2^-24 covers the rounding of those that are
    const double inv = 1.0 / (double)cand;
    uint32_t columns = (uint32_t)(b.n_live - n_long), blocks = 0;  // blocks: of sums that a reduction pass moves
    for (int i = 0; i < n_long; ++i) {
      const uint32_t w = (uint32_t)((int32_t)((double)(int32_t)(longer[i] + cand - 1) * inv + 0x1p-24));
      columns += w;
      blocks += w > 1 ? 2 * w + 1 : 0;
    }
    if ((int64_t)columns > budget + b.n_live) return;  // (the bound that the scratch is sized by)
    const int64_t per_cu = ((int64_t)columns * n_tiles + cus - 1) / cus;  // workgroups of the fullest CU
    double cost = (double)cand * (per_cu < wg_per_cu ? share[per_cu] : 1.0) + kBatchColumnEpochs;
    if ((int64_t)columns > budget) {
      const double dealt =
          ((double)total_epochs + kBatchColumnEpochs * (double)columns) / (double)budget + 0.5 * (double)cand;
      if (dealt > cost) cost = dealt;
    }
    if (blocks) cost += kBatchMergeLaunchEpochs + kBatchMergeEpochs * (double)blocks / (double)budget;
    if (cost < t_cost) {
      t_cost = cost;
      t = cand;
    }
  };
  if (n_long > 0) {  // (else every leaf has one column whatever T is)
    const double alone = wg_per_cu <= 2 ? kBatchAloneShareOfTwo : kBatchAloneShare;
    for (int k = 1; k < wg_per_cu && k < kBatchMaxPerCu; ++k)
      share[k] = alone + (1.0 - alone) * (double)k / (double)wg_per_cu;
    consider(most);
    auto consider_around = [&](int64_t columns, std::initializer_list<double> factors) {
      const double average = (double)total_epochs / (double)columns;
      for (const double factor : factors) {
        const double cand = std::ceil(average * factor);
        if (cand < (double)most) consider(cand < 1.0 ? 1u : (uint32_t)cand);
      }
    };
    consider_around(budget, {0.4, 0.45, 0.5, 0.55, 0.65, 0.8, 1.0, 1.03, 1.1, 1.25, 1.5, 2.0, 4.0});
    for (int k = 1; k < wg_per_cu && k < kBatchMaxPerCu; ++k)
      if ((int64_t)k * cus >= n_tiles) consider_around((int64_t)k * cus / n_tiles, {1.0, 1.03, 1.1, 1.25});
  }
  int wgs[kBatchLeaves], unit[kBatchLeaves];
  uint32_t each[kBatchLeaves];  // epochs of a leaf's busiest workgroup
  for (int i = 0; i < n; ++i) {
    if (epochs[i] <= (uint32_t)kDirectEpochs) {  // (as plan_leaf_units has it)
      wgs[i] = epochs[i] > 0;
      unit[i] = epochs[i] > 0 ? (int)epochs[i] : 1;
      each[i] = epochs[i];
    } else {
      bool one_each = false;
      plan_leaf_units((int64_t)epochs[i], (int64_t)((epochs[i] + t - 1) / t), &wgs[i], &unit[i], &one_each);
      each[i] = one_each ? (uint32_t)unit[i] : (epochs[i] + (uint32_t)wgs[i] - 1) / (uint32_t)wgs[i];
    }
    if (each[i] > b.most_each) b.most_each = each[i];
    if (unit[i] > b.most_unit_epochs) b.most_unit_epochs = unit[i];
  }
  // the longest first, to within 1/128 of the longest (equal ones in the call's order): a counting sort,
  // because a call of many short leaves takes about as long on the host as on the device
  int shift = 0;
  while ((b.most_each >> shift) > 255u) ++shift;
  uint16_t place[257] = {0};  // place[k + 1] ends as the first place of key k, keys descending
  for (int i = 0; i < n; ++i) ++place[256 - (each[i] >> shift)];
  for (int k = 1; k <= 256; ++k) place[k] = (uint16_t)(place[k] + place[k - 1]);
  int order[kBatchLeaves];
  for (int i = 0; i < n; ++i) order[place[255 - (each[i] >> shift)]++] = i;
  uint32_t first = 0;
  for (int k = 0; k < n; ++k) {
    const int i = order[k];
    b.leaf[k].row_off =
        seg_off ? seg_off[l0 + i] : (uint32_t)(leaf_offsets[l0 + i] - leaf_offsets[l0]);
    b.leaf[k].n = (uint32_t)(leaf_offsets[l0 + i + 1] - leaf_offsets[l0 + i]);
    b.leaf[k].first_wg = first;
    b.leaf[k].packed = batch_leaf_pack((uint32_t)wgs[i], (uint32_t)unit[i], (uint32_t)i);
    first += (uint32_t)wgs[i];
  }
  b.total_wgs = first;
  return b;
}

// Which of its two kernels a batch takes (see leaf_is_short).  Leaves of about one column end where their workgroup does, which writes the
// histogram: SHORT, unless there are many epochs before that.  With two columns a leaf and more most workgroups end elsewhere.
// One column, SHORT and long us: a tenth of 1,500,000 x 500 x 255 in 64 leaves, 5 epochs, 61.7 and 71.8, all of it in 128, 23 epochs, 394.6 and
// 405.7, in 64, 46 epochs, 351.4 and 354.2, in 32, 92 epochs, 304.4 and 302.0, in 24, 123 epochs, 383.2 and 378.1; half of 400,000 x 2,000 x 63 in
// 128, 4 epochs, 164.7 and 180.9; half of 8,000,000 x 500 x 64 in 128, 62 epochs, 751 and 716.
// More: a tenth of 1,500,000 x 500 x 255 in four, eight columns of 10 epochs, 57.7 and 56.7, all of it in 16, two of 92, 315.9 and 310.4; 30 % of
// 2,270,000 x 137 x 255 in 20, five of 14, 82.7 and 81.2; 10,500,000 x 28 x 255 in one, 41 epochs, 151.3 and 147.3, in 64, the same, 234; a tenth of
// 10,500,000 x 60 x 64 in 128 with wide sums 68.6 and 67.7, without 0 to 1 % either way.  (The other way round where equal leaves take every place there
// is: 10,500,000 x 28 x 255 in 16, 32 columns each, 183 and 189.)
// With 16 bins there is nothing between the two but on one column, where SHORT gains 1 to 5 %; wide 256 bins have one kernel.
constexpr uint32_t kBatchLongEpochs = 60;
bool batch_is_short(const BatchPlan& b, int cap, bool wide) {
  if (!batch_has_long(cap, wide)) return true;
  return b.total_wgs < 2u * (uint32_t)b.n_live && b.most_each <= kBatchLongEpochs;
}

// The table of one launch of stats_gather_lists_kernel, for lists l0, l0 + 1, ... of the call: as many as fit the table, and
// as start within 2^32 positions of list l0 (each is shorter than 2^31).  Without seg_off positions are relative to list l0's.
// Returns the blocks of an eighth of the lists.
uint32_t fill_gather_table(const int64_t* leaf_offsets, const uint32_t* seg_off, int32_t l0, int32_t n_leaves,
                           GatherTable* t) {
  uint32_t blocks = 0;
  int32_t i = 0;
  for (; i < kGatherLists && l0 + i < n_leaves; ++i) {
    const int64_t n = leaf_offsets[l0 + i + 1] - leaf_offsets[l0 + i];
    if (!seg_off && leaf_offsets[l0 + i + 1] - leaf_offsets[l0] >= ((int64_t)1 << 32)) break;
    t->first[i] = seg_off ? seg_off[l0 + i] : (uint32_t)(leaf_offsets[l0 + i] - leaf_offsets[l0]);
    t->n[i] = (uint32_t)n;
    t->first_block[i] = blocks;
    blocks += (uint32_t)(((n + kXcds - 1) / kXcds + kGatherRows - 1) / kGatherRows);
  }
  t->n_lists = i;
  return blocks;
}

// Split search of n_hists (<= kSplitMaxHists) histograms, hist_stride bins apart, in one
// launch; splits_out[i] receives the record of histogram i.
int launch_split(const gbdt_bin_t* hists, int64_t hist_stride, int32_t n_hists, float lambda,
                 float min_child_hess, gbdt_split_t* splits_out, int32_t n_features, int32_t n_bins,
                 hipStream_t s, gbdt_split_t* mirror = nullptr, const SplitSiblings* siblings = nullptr) {
  const SplitGrouping sg = split_grouping(n_features, n_bins, n_hists);
  void* ws = nullptr;
  if (sg.n_wg > 1) {  // (a lone workgroup hands nothing over)
    const int rc = get_workspace((size_t)n_hists * sg.n_wg * sizeof(SplitCand), s, &ws);
    if (rc != GBDT_OK) return rc;
  }
  // (only with siblings does the kernel write to the histograms)
  auto launch = [&](auto kernel, const auto& sib) {
    hipLaunchKernelGGL(kernel, dim3(sg.n_wg, n_hists), dim3(64 * sg.waves), 0, s, const_cast<gbdt_bin_t*>(hists),
                       hist_stride, n_features, n_bins, sg.passes, (double)lambda, (double)min_child_hess,
                       (SplitCand*)ws, splits_out, mirror, sib);
  };
  auto launch_of = [&](const auto& sib) {
    using SIB = std::decay_t<decltype(sib)>;
    switch (n_bins < kSplitBins ? 0 : split_lane_bits(n_bins)) {
      case 0: launch(split_gain_kernel<2, true, SIB>, sib); break;
      case 2: launch(split_gain_kernel<2, false, SIB>, sib); break;
      case 3: launch(split_gain_kernel<3, false, SIB>, sib); break;
      case 4: launch(split_gain_kernel<4, false, SIB>, sib); break;
      case 5: launch(split_gain_kernel<5, false, SIB>, sib); break;
      default: launch(split_gain_kernel<6, false, SIB>, sib); break;
    }
  };
  if (siblings) {
    launch_of(*siblings);
  } else {
    launch_of(NoSiblings{});
  }
  HIP_TRY(hipGetLastError());
  return GBDT_OK;
}

// Scratch of gbdt_grow_tree.
size_t align256(size_t b) { return (b + 255) / 256 * 256; }

// gbdt_grow_tree expands up to kGrowRound open leaves per round (one wait for the stream per
// round instead of one per split) and may expand leaves that best-first growth never gets to
// before the leaf budget is used up; the histogram pool is sized for the splits of the tree plus
// that many speculative ones.
constexpr int kGrowRound = 32;
static_assert(kGrowRound <= kSplitSiblings, "a round's siblings travel as one kernel argument");
int32_t grow_speculative_budget(int32_t max_leaves) { return (max_leaves - 1) / 2 + 16; }
int32_t grow_max_expansions(int32_t max_leaves) { return (max_leaves - 1) + grow_speculative_budget(max_leaves); }

struct TreeScratch {
  size_t rows_a, rows_b, hists, recs;  // byte offsets
  size_t pairs;       // (gradient, hessian) of every row; only where they pay
  size_t least;       // bytes without the pairs: a caller's scratch of that size still serves
  size_t total;
  size_t row_elems;   // int32 entries between the two row buffers
  int32_t n_slots;    // histograms in the pool
};

TreeScratch tree_scratch_layout(int64_t n_rows, int32_t n_features, int32_t n_bins, int32_t max_leaves) {
  TreeScratch t;
  const size_t rows = align256((size_t)(n_rows > 0 ? n_rows : 1) * sizeof(int32_t));
  t.row_elems = rows / sizeof(int32_t);
  t.n_slots = 1 + 2 * grow_max_expansions(max_leaves);
  t.rows_a = 0;
  t.rows_b = rows;
  t.hists = 2 * rows;
  t.recs = t.hists + align256((size_t)t.n_slots * n_features * n_bins * sizeof(gbdt_bin_t));
  t.pairs = t.least = t.recs + align256((size_t)t.n_slots * sizeof(gbdt_split_t));
  t.total = t.least + (stats_pair_pays(plan_n_tiles(make_tile_plan(n_features, n_bins)), n_rows)
                           ? align256((size_t)n_rows * sizeof(float2)) : 0);
  return t;
}

// Page-locked host memory for the split records of a round or level, which the split search writes there as well as to device
// memory: the host reads them after waiting for the stream, without a copy (20,000 x 30 x 64 to depth 5, which read them back
// and sent the partition's copies of them: 258 us, 203 so).  A grower borrows a block for the length of its call, so growers of
// several threads never share one; up to kIdleRecordBlocks are kept for later calls, until gbdt_reset.
constexpr size_t kIdleRecordBlocks = 4;
struct RecordBlock {
  gbdt_split_t *host, *dev;  // the same memory, as the host and as the device addresses it
  size_t n;
  int device;
};
struct RecordBlocks {
  std::mutex mu;
  std::vector<RecordBlock> idle, lost;  // lost: a kernel that failed calls left behind may still write to it
} g_rec_blocks;
class HostRecords {
 public:
  explicit HostRecords(size_t n) {
    b_ = RecordBlock{nullptr, nullptr, 512, 0};
    if (hipGetDevice(&b_.device) != hipSuccess) return;
    std::lock_guard<std::mutex> lk(g_rec_blocks.mu);
    auto& idle = g_rec_blocks.idle;
    for (size_t i = 0; i < idle.size(); ++i) {
      if (idle[i].device != b_.device || idle[i].n < n) continue;
      b_ = idle[i];
      idle.erase(idle.begin() + (ptrdiff_t)i);
      return;
    }
    while (b_.n < n) b_.n *= 2;
    void *q = nullptr, *dq = nullptr;
    if (hipHostMalloc(&q, b_.n * sizeof(gbdt_split_t), hipHostMallocMapped) != hipSuccess) {
      (void)hipGetLastError();
      return;
    }
    if (hipHostGetDevicePointer(&dq, q, 0) != hipSuccess) {
      (void)hipGetLastError();
      (void)hipHostFree(q);
      return;
    }
    b_.host = (gbdt_split_t*)q;
    b_.dev = (gbdt_split_t*)dq;
  }
  ~HostRecords() {
    if (!b_.host) return;
    std::lock_guard<std::mutex> lk(g_rec_blocks.mu);
    if (!in_flight_ && g_rec_blocks.idle.size() >= kIdleRecordBlocks) {
      // the largest are kept: a small one serves fewer calls, and allocating and freeing takes longer than most calls
      auto least = std::min_element(g_rec_blocks.idle.begin(), g_rec_blocks.idle.end(),
                                    [](const RecordBlock& x, const RecordBlock& y) { return x.n < y.n; });
      if (least->n < b_.n) std::swap(*least, b_);
      (void)hipHostFree(b_.host);
      return;
    }
    try {
      (in_flight_ ? g_rec_blocks.lost : g_rec_blocks.idle).push_back(b_);
    } catch (...) {  // (no memory for the list: the block is not seen again)
    }
  }
  HostRecords(const HostRecords&) = delete;
  HostRecords& operator=(const HostRecords&) = delete;
  bool ok() const { return b_.host != nullptr; }
  const gbdt_split_t& operator[](size_t i) const { return b_.host[i]; }
  gbdt_split_t* device() { return b_.dev; }  // for the call that enqueues a kernel
  // ... and what that call returned: without the scratch it needs it has enqueued nothing, and nobody writes to the block
  int enqueued(int rc) {
    in_flight_ = in_flight_ || rc != GBDT_ENOMEM;
    return rc;
  }
  // the block as words, of which it holds at least n * sizeof(gbdt_split_t) / 4
  uint32_t* device_words() { return reinterpret_cast<uint32_t*>(b_.dev); }
  const uint32_t* words() const { return reinterpret_cast<const uint32_t*>(b_.host); }
  hipError_t wait(hipStream_t s) {  // until the kernels that write to the block are done
    const hipError_t e = hipStreamSynchronize(s);
    if (e == hipSuccess) in_flight_ = false;
    return e;
  }

 private:
  RecordBlock b_;
  bool in_flight_ = false;
};

// A split that sends more rows to the children than the node has cannot be: the rows of the children would not be the node's.
bool split_fits(const gbdt_split_t& r, uint64_t count) {
  if (r.feature < 0 || (uint64_t)r.left_count + r.right_count <= count) return true;
  snprintf(g_hip_err, sizeof g_hip_err, "a split of %u and %u rows was found for a node of %llu", r.left_count, r.right_count,
           (unsigned long long)count);
  return false;
}

// Scratch of gbdt_grow_tree_depthwise: two row buffers, two levels of histograms and the split records of a level.
constexpr int kMaxTreeDepth = 16;
struct LevelScratch {
  size_t rows_a, rows_b, hists_a, hists_b, recs, total;
};

LevelScratch level_scratch_layout(int64_t n_rows, int32_t n_features, int32_t n_bins, int32_t max_depth) {
  LevelScratch t;
  const size_t rows = align256((size_t)(n_rows > 0 ? n_rows : 1) * sizeof(int32_t));
  const size_t width = (size_t)1 << max_depth;
  const size_t hists = align256(width * n_features * n_bins * sizeof(gbdt_bin_t));
  const size_t recs = align256(width * sizeof(gbdt_split_t));
  t.rows_a = 0;
  t.rows_b = rows;
  t.hists_a = 2 * rows;
  t.hists_b = t.hists_a + hists;
  t.recs = t.hists_b + hists;
  t.total = t.recs + recs;
  return t;
}

// gbdt_hist_build, with the scratch either the library's workspace (fixed_base == NULL) or a
// fixed buffer of fixed_bytes whose head holds the unit counters (the no-allocation entry
// point): then nothing is allocated, the grid shrinks until its partial blocks fit, and
// the counters are zeroed by every call that uses them.
int hist_build_impl(const void* bin_matrix, int64_t n_rows, int32_t n_features, int32_t n_bins,
                    const int32_t* leaf_row_idx, int64_t n_leaf_rows, const float* grad,
                    const float* hess, gbdt_bin_t* hist_out, void* stream, void* fixed_base,
                    size_t fixed_bytes) {
  g_hip_err[0] = 0;
  if (!valid_shape(n_rows, n_features, n_bins)) return GBDT_EINVAL;
  if (!hist_out) return GBDT_EINVAL;
  if (n_leaf_rows < 0) return GBDT_EINVAL;
  if (!leaf_row_idx && n_leaf_rows > n_rows) return GBDT_EINVAL;
  if (n_rows >= ((int64_t)1 << 30) || n_leaf_rows >= ((int64_t)1 << 31)) return GBDT_EUNSUPPORTED;
  hipStream_t s = (hipStream_t)stream;
  if (n_leaf_rows == 0) {
    const int32_t n = n_features * n_bins;
    hipLaunchKernelGGL(hist_zero_kernel, dim3((n + 255) / 256), dim3(256), 0, s, hist_out, n);
    HIP_TRY(hipGetLastError());
    return GBDT_OK;
  }
  if (!bin_matrix || !grad || !hess) return GBDT_EINVAL;
  if (!fixed_base) {  // (the checking kernel's counter lives in the library's workspace)
    const int rc_ids = check_row_ids(leaf_row_idx, n_leaf_rows, n_rows, s);
    if (rc_ids != GBDT_OK) return rc_ids;
  }

  const bool wide = g_wide.load() != 0;
  // A fused copy of the matrix (few-level features sharing columns): the build kernel then sees
  // build_f one-byte columns of kFusedCap joint bins, and the marginals are taken at the end.
  FusedEntry fe;
  // (not with wide accumulation: the joint histograms are rounded to fp32 before the marginals are
  // taken, which would break that mode's promise of the exact sum rounded once)
  const bool fused = !wide && n_leaf_rows >= kFusedMinLeafRows && n_leaf_rows * kFusedMinLeafFraction >= n_rows &&
                     fused_lookup(bin_matrix, n_rows, n_features, n_bins, &fe);
  const int32_t real_features = n_features, real_bins = n_bins;
  if (fused) {
    n_features = fe.n_cols;
    n_bins = kFusedCap;
  }
  const size_t joint_words = fused ? (size_t)n_features * n_bins * 3 : 0;
  const TilePlan plan0 = make_tile_plan(n_features, n_bins);
  const bool halves = plan_halves(plan0, wide, rows_of_leaf(leaf_row_idx != nullptr, n_leaf_rows, n_rows));
  const int wg_per_cu = build_wg_per_cu(plan0.cap, leaf_row_idx != nullptr, wide, halves);
  BuildGeom g = make_geom(n_features, n_bins, n_leaf_rows, device_cu_count(), wg_per_cu, wide, halves);
  if (fixed_base) {
    // fewer workgroups per tile until the partial blocks fit the fixed buffer
    size_t avail_words = fixed_bytes > kWsHeadBytes ? (fixed_bytes - kWsHeadBytes) / 4 : 0;
    avail_words = avail_words > joint_words ? avail_words - joint_words : 0;
    if (g.partial_words > avail_words) {
      const size_t per_wg = g.partial_words / (size_t)g.wgs;  // words of one workgroup of every tile
      const int64_t fit = (int64_t)(avail_words / per_wg);
      if (fit < 1) {
        snprintf(g_hip_err, sizeof g_hip_err,
                 "%d features x %d bins need %zu bytes of partial histograms, the fixed scratch holds %zu",
                 n_features, n_bins, per_wg * 4, avail_words * 4);
        return GBDT_EUNSUPPORTED;
      }
      g = make_geom(n_features, n_bins, n_leaf_rows, device_cu_count(), wg_per_cu, wide, halves, fit);
    }
  }
  const TilePlan& p = g.plan;
  if (plan_n_tiles(p) > 65535) return GBDT_EUNSUPPORTED;
  // byte offsets inside a tile (slack included) are formed in 32 bits
  if ((n_rows + kEpochRows) * (int64_t)p.wm >= ((int64_t)1 << 32)) return GBDT_EUNSUPPORTED;
  const int32_t line_tiles = fused ? 1 : plan_line_tiles(n_rows);  // (a fused copy has a region per tile)
  void* ws = nullptr;
  uint32_t* counters = nullptr;
  bool counters_zero = false;
  // With an index list and several feature tiles, gather grad / hess into leaf order once
  // instead of letting every tile's workgroups gather them from scattered rows.
  bool by_pos = leaf_row_idx != nullptr && stats_gather_pays(plan_n_tiles(p), n_leaf_rows, n_leaf_rows, n_rows);
  size_t stats_words = by_pos ? 2 * (((size_t)n_leaf_rows + 63) / 64 * 64) : 0;
  int rc = GBDT_OK;
  if (fixed_base) {
    if (kWsHeadBytes + (g.partial_words + joint_words + stats_words) * 4 > fixed_bytes) {  // the gather is optional
      by_pos = false;
      stats_words = 0;
    }
    counters = (uint32_t*)fixed_base;
    ws = (char*)fixed_base + kWsHeadBytes;
    counters_zero = false;
  } else {
    rc = get_workspace((g.partial_words + joint_words + stats_words) * 4, s, &ws, &counters, &counters_zero);
    if (rc == GBDT_ENOMEM && by_pos) {  // a caller's workspace sized for the partial blocks alone: no gather
      by_pos = false;
      stats_words = 0;
      rc = get_workspace((g.partial_words + joint_words) * 4, s, &ws, &counters, &counters_zero);
    }
  }
  if (rc != GBDT_OK) return rc;

  // scratch: [partial blocks][joint histograms of the fused columns][grad / hess in leaf order]
  gbdt_bin_t* joint = (gbdt_bin_t*)((uint32_t*)ws + g.partial_words);
  BuildArgs a;
  a.packed = fused ? fe.tiles : (const uint8_t*)bin_matrix;
  a.idx = leaf_row_idx;
  a.grad = grad;
  a.hess = hess;
  a.stats_by_pos = 0;
  if (by_pos) {
    float* g_leaf = (float*)ws + g.partial_words + joint_words;
    float* h_leaf = g_leaf + stats_words / 2;
    hipLaunchKernelGGL(stats_gather_kernel, dim3((unsigned)((n_leaf_rows + 255) / 256)), dim3(256), 0, s,
                       leaf_row_idx, grad, hess, n_leaf_rows, g_leaf, h_leaf);
    HIP_TRY(hipGetLastError());
    a.grad = g_leaf;
    a.hess = h_leaf;
    a.stats_by_pos = 1;
  }
  a.partials = (uint32_t*)ws;
  a.counters = counters;
  a.n_rows = n_rows;
  a.n_leaf = n_leaf_rows;
  a.n_main = p.n_main;
  a.wr = p.wr;
  a.line_tiles = line_tiles;
  a.wgs = g.wgs;
  a.chunks = g.wgs * g.blocks_per_wg;
  const UnitPlan u = plan_units(g, n_leaf_rows, leaf_row_idx != nullptr, line_tiles, g_deterministic.load(), device_cu_count());
  a.unit_epochs = u.unit_epochs;
  a.first_epochs = u.first_epochs;
  a.fixed_stride = u.fixed_stride;
  a.deal = u.deal;
  a.direct_out = (g.wgs == 1 && !fused) ? hist_out : nullptr;  // (joint histograms always take the reduction pass)
  a.n_features = n_features;
  a.n_bins = n_bins;
  const int blocks = g.parts * g.wgs;
  const bool uses_counters = a.fixed_stride == 0;
  // While the stream is being captured nothing runs now, so what is known about the
  // counters must not change: the captured sequence zeroes them itself, before and (if
  // no reduction pass follows) after the build, and leaves them zero on every replay.
  // (the fixed buffer is treated the same way: what is known about it is not tracked)
  const bool capturing = fixed_base != nullptr || stream_is_capturing(s);
  auto zero_counters = [&]() -> int {
    hipLaunchKernelGGL(counters_zero_kernel, dim3(kCounterSlots / 256), dim3(256), 0, s, counters,
                       kCounterSlots);
    HIP_TRY(hipGetLastError());
    return GBDT_OK;
  };
  if (uses_counters && (capturing || !counters_zero)) {  // e.g. a new scratch buffer
    rc = zero_counters();
    if (rc != GBDT_OK) return rc;
  }
  // From here until the reduction pass has been enqueued the counters are in use.
  if (uses_counters && !capturing) set_counters_zero(counters, false);

  const bool is_short = leaf_is_short(g, wide);
  const bool timed = fixed_base == nullptr;  // the profiling events are created on the fly: an allocation
  if (wide) {
    if (p.cap == 16) {
      rc = launch_build<GBDT_VARIANT_16W, true>(a, blocks, s, timed, is_short);
    } else if (p.cap == 64) {
      rc = launch_build<GBDT_VARIANT_64W, true>(a, blocks, s, timed, is_short);
    } else if (halves) {
      rc = launch_build<GBDT_VARIANT_256W_HALVES, true, true>(a, blocks, s, timed, is_short);
    } else {
      rc = launch_build<GBDT_VARIANT_256W, true, false, true>(a, blocks, s, timed, is_short);
    }
  } else if (p.cap == 16) {
    rc = launch_build<GBDT_VARIANT_16>(a, blocks, s, timed, is_short);
  } else if (p.cap == 64) {
    rc = launch_build<GBDT_VARIANT_64>(a, blocks, s, timed, is_short);
  } else {
    rc = launch_build<GBDT_VARIANT_256>(a, blocks, s, timed, is_short);
  }
  if (rc != GBDT_OK) return rc;
  if (a.direct_out) {  // one workgroup per tile: the histogram is written
    if (uses_counters && capturing) return zero_counters();
    return GBDT_OK;
  }

  MergeArgs m;
  m.partials = (const uint32_t*)ws;
  m.out = fused ? joint : hist_out;
  m.plan = p;
  m.n_features = n_features;
  m.n_bins = n_bins;
  m.chunks_main = a.chunks;
  m.chunks_rem = p.wr ? a.chunks : 0;
  m.halves = halves ? 1 : 0;
  m.counters = uses_counters ? counters : nullptr;
  const int64_t tile_cells = merge_tile_cells(p, n_bins);
  const int parts = merge_parts(tile_cells, plan_n_tiles(p), a.chunks);
  const dim3 merge_grid((unsigned)((tile_cells + merge_wg_cells(parts) - 1) / merge_wg_cells(parts)), plan_n_tiles(p));
  auto merge = [&](auto kernel) { hipLaunchKernelGGL(kernel, merge_grid, dim3(merge_wg_threads(parts)), 0, s, m); };
  merge(parts == 1 ? hist_merge_kernel<1> : parts == 2 ? hist_merge_kernel<2> : parts == 4 ? hist_merge_kernel<4>
        : parts == kMergePartsMost ? hist_merge_kernel<kMergePartsMost> : hist_merge_kernel<kMergePartsWide>);
  HIP_TRY(hipGetLastError());
  if (uses_counters && !capturing) set_counters_zero(counters, true);  // the reduction pass leaves them zero
  if (fused) {
    const int32_t n = real_features * real_bins;
    hipLaunchKernelGGL(hist_unfuse_kernel, dim3((n + 255) / 256), dim3(256), 0, s, (const gbdt_bin_t*)joint, fe.feats,
                       real_features, real_bins, hist_out);
    HIP_TRY(hipGetLastError());
  }
  return GBDT_OK;
}


}  // namespace

// ----------------------------------------------------------------------- C ABI

extern "C" {

size_t gbdt_bins_packed_bytes(int64_t n_rows, int32_t n_features, int32_t n_bins) {
  if (!valid_shape(n_rows, n_features, n_bins)) return 0;
  const TilePlan p = make_tile_plan(n_features, n_bins);
  return (size_t)plan_packed_bytes(p, n_rows, n_features);
}

int gbdt_bins_pack(const uint8_t* bins_rowmajor, int64_t n_rows, int32_t n_features,
                   int32_t n_bins, void* packed_out, void* stream) {
  if (!valid_shape(n_rows, n_features, n_bins)) return GBDT_EINVAL;
  if (packed_out) (void)gbdt_bins_unfuse(packed_out);  // a fused copy registered for this address is stale now
  if (n_rows == 0) return GBDT_OK;
  if (!bins_rowmajor || !packed_out) return GBDT_EINVAL;
  if (((uintptr_t)packed_out & 15u) != 0) return GBDT_EINVAL;
  if (n_rows >= ((int64_t)1 << 31)) return GBDT_EUNSUPPORTED;
  const TilePlan p = make_tile_plan(n_features, n_bins);
  const int tiles = plan_n_tiles(p);
  if (tiles > 65535) return GBDT_EUNSUPPORTED;
  if ((n_features + 63) / 64 > 65535) return GBDT_EUNSUPPORTED;
  const dim3 grid((unsigned)((n_rows + kPackRows - 1) / kPackRows),
                  (unsigned)((n_features + kPackFeatures - 1) / kPackFeatures));
  const bool big = plan_packed_bytes(p, n_rows, n_features) > kPackStreamBytes;
  const auto kernel = p.nib ? (big ? pack_kernel<true, true> : pack_kernel<true, false>)
                            : (big ? pack_kernel<false, true> : pack_kernel<false, false>);
  hipLaunchKernelGGL(kernel, grid, dim3(256), 0, (hipStream_t)stream, bins_rowmajor, n_rows, n_features, p, plan_line_tiles(n_rows),
                     (uint32_t)(p.cap - 1) * 0x01010101u, (uint8_t*)packed_out,
                     (uint8_t*)packed_out + plan_columns_base(p, n_rows), plan_column_stride(n_rows));
  HIP_TRY(hipGetLastError());
  return GBDT_OK;
}

size_t gbdt_bins_fused_bytes(int64_t n_rows, int32_t n_features, int32_t n_bins) {
  if (!valid_shape(n_rows, n_features, n_bins) || n_bins > kFusedCap || n_rows == 0) return 0;
  const int32_t max_cols = (int32_t)(kFusedMaxColumnRatio * n_features);
  if (max_cols < 1) return 0;
  return fused_layout(n_rows, n_features, max_cols).total;
}

int gbdt_bins_unfuse(const void* packed) {
  std::lock_guard<std::mutex> lk(g_fused_mu);
  g_fused.erase(packed);
  return GBDT_OK;
}

int gbdt_bins_fuse(const uint8_t* bins_rowmajor, int64_t n_rows, int32_t n_features, int32_t n_bins,
                   const void* packed, void* fused_out, size_t fused_bytes, int32_t* n_columns_out,
                   void* stream) {
  g_hip_err[0] = 0;
  if (!valid_shape(n_rows, n_features, n_bins) || !n_columns_out || !packed) return GBDT_EINVAL;
  *n_columns_out = 0;
  (void)gbdt_bins_unfuse(packed);
  if (n_bins > kFusedCap || n_rows == 0) return GBDT_OK;  // never fused
  if (!bins_rowmajor || !fused_out) return GBDT_EINVAL;
  if (((uintptr_t)fused_out & 255u) != 0) return GBDT_EINVAL;
  if (fused_bytes < (size_t)n_features * sizeof(uint32_t)) return GBDT_ENOMEM;
  if (n_rows >= ((int64_t)1 << 30)) return GBDT_EUNSUPPORTED;
  hipStream_t s = (hipStream_t)stream;
  if (stream_is_capturing(s)) return GBDT_EUNSUPPORTED;  // this call reads results on the host
  // 1. the largest bin value of every feature (the head of fused_out serves as scratch).  First over the
  // first kFuseSampleRows rows: columns hold at most log2(kFusedCap) bits, so features that need more
  // bits than kFusedMaxColumnRatio of that many columns have -- with the levels seen so far, which can
  // only grow -- are never fused, and the rest of the matrix need not be read to know it.
  uint32_t* max_dev = (uint32_t*)fused_out;
  hipLaunchKernelGGL(counters_zero_kernel, dim3((n_features + 255) / 256), dim3(256), 0, s, max_dev, n_features);
  HIP_TRY(hipGetLastError());
  if ((n_rows + 255) / 256 >= ((int64_t)1 << 31)) return GBDT_EUNSUPPORTED;
  std::vector<uint32_t> levels((size_t)n_features);
  // A kernel writes the maxima to page-locked memory: a copy to the vector goes through the runtime's staging buffer
  // and a kernel of its own (10,000 x 28 x 64 packed in 35.1 us so, 28.6 this way; 20,000 x 700 x 16 60.2 and 52.5; pack, root,
  // split and rows of 400,000 x 2,000 x 63 725 and 700).  Without page-locked memory that copy is made.
  HostRecords found(((size_t)n_features * sizeof(uint32_t) + sizeof(gbdt_split_t) - 1) / sizeof(gbdt_split_t));
  auto find_levels = [&](int64_t rows) -> int {
    int32_t lane_bits = 0;  // threads across a row, 16 features each
    while (lane_bits < 6 && (16 << lane_bits) < n_features) ++lane_bits;
    const int64_t block_rows = (int64_t)(256 >> lane_bits) * kMaxFlight;
    const int64_t stripes = (rows + block_rows - 1) / block_rows;
    const int64_t most = rows >= kFuseSampleMinRows ? 1024 : 64;  // (every workgroup ends with atomics)
    hipLaunchKernelGGL(feature_max_kernel,
                       dim3((unsigned)(stripes < most ? stripes : most),
                            (unsigned)((n_features + kMaxFeatures - 1) / kMaxFeatures)),
                       dim3(256), 0, s, bins_rowmajor, rows, n_rows, n_features, lane_bits, max_dev);
    HIP_TRY(hipGetLastError());
    if (found.ok()) {
      hipLaunchKernelGGL(words_copy_kernel, dim3((n_features + 255) / 256), dim3(256), 0, s, (const uint32_t*)max_dev,
                         n_features, found.device_words());
      (void)found.enqueued(GBDT_OK);
      HIP_TRY(hipGetLastError());
      HIP_TRY(found.wait(s));
      std::copy(found.words(), found.words() + n_features, levels.begin());
    } else {
      HIP_TRY(hipMemcpyAsync(levels.data(), max_dev, levels.size() * sizeof(uint32_t), hipMemcpyDeviceToHost, s));
      HIP_TRY(hipStreamSynchronize(s));
    }
    for (uint32_t& l : levels) {
      l = l + 1;                       // bins 0 .. max occur (at most)
      if (l > (uint32_t)n_bins) l = (uint32_t)n_bins;  // the build masks stray values to the capacity anyway
    }
    return GBDT_OK;
  };
  if (const int64_t sample = fuse_sample_rows(n_rows, n_features)) {
    const int rc = find_levels(sample);
    if (rc != GBDT_OK) return rc;
    double bits = 0.0;
    for (const uint32_t l : levels) bits += std::log2((double)l);
    // (a thousandth of a bit a feature to spare for the rounding of the logarithms)
    if (bits - 1e-3 * n_features > kFusedMaxColumnRatio * n_features * std::log2((double)kFusedCap)) return GBDT_OK;
  }
  const int rc_levels = find_levels(n_rows);
  if (rc_levels != GBDT_OK) return rc_levels;
  // 2. the plan; does it pay?
  std::vector<FusedCol> cols;
  std::vector<FusedFeat> feats;
  plan_fusion(levels, &cols, &feats);
  const int32_t n_cols = (int32_t)cols.size();
  if ((double)n_cols > kFusedMaxColumnRatio * n_features) return GBDT_OK;
  const FusedLayout lay = fused_layout(n_rows, n_features, n_cols);
  if (lay.total > fused_bytes) {
    snprintf(g_hip_err, sizeof g_hip_err, "fused copy needs %zu bytes, %zu given", lay.total, fused_bytes);
    return GBDT_ENOMEM;
  }
  if (plan_n_tiles(lay.plan) > 65535) return GBDT_OK;
  // 3. tables, then the tiles
  char* base = (char*)fused_out;
  HIP_TRY(hipMemcpyAsync(base + lay.feats_off, feats.data(), feats.size() * sizeof(FusedFeat), hipMemcpyHostToDevice, s));
  HIP_TRY(hipMemcpyAsync(base + lay.cols_off, cols.data(), cols.size() * sizeof(FusedCol), hipMemcpyHostToDevice, s));
  const int tiles = plan_n_tiles(lay.plan);
  const int64_t max_words = n_rows * (lay.plan.wm / 4);
  const int64_t bx = (max_words + 255) / 256;
  if (bx >= ((int64_t)1 << 31)) return GBDT_EUNSUPPORTED;
  const FusedCol* cols_dev = (const FusedCol*)(base + lay.cols_off);
  if (n_features <= kFuseStageFeatures) {
    hipLaunchKernelGGL(pack_fused_staged_kernel, dim3((unsigned)((n_rows + kFuseStageRows - 1) / kFuseStageRows)),
                       dim3(256), (size_t)kFuseStageRows * n_features, s, bins_rowmajor, n_rows, n_features, lay.plan,
                       cols_dev, n_cols, (uint8_t*)base);
  } else {
    hipLaunchKernelGGL(pack_fused_kernel, dim3((unsigned)bx, (unsigned)tiles), dim3(256), 0, s, bins_rowmajor, n_rows,
                       n_features, lay.plan, cols_dev, n_cols, (uint8_t*)base);
  }
  HIP_TRY(hipGetLastError());
  HIP_TRY(hipStreamSynchronize(s));  // the host tables must outlive their copies
  FusedEntry e;
  e.tiles = (const uint8_t*)base;
  e.feats = (const FusedFeat*)(base + lay.feats_off);
  e.n_rows = n_rows;
  e.n_features = n_features;
  e.n_bins = n_bins;
  e.n_cols = n_cols;
  {
    std::lock_guard<std::mutex> lk(g_fused_mu);
    g_fused[packed] = e;
  }
  *n_columns_out = n_cols;
  return GBDT_OK;
}

size_t gbdt_workspace_bytes(int64_t n_rows, int32_t n_features, int32_t n_bins) {
  if (!valid_shape(n_rows, n_features, n_bins)) return 0;
  const int cap = make_tile_plan(n_features, n_bins).cap;
  const bool wide = g_wide.load() != 0;
  // (a list that is built from whole tiles has half the resident workgroups and needs as much)
  const bool halves = plan_halves(make_tile_plan(n_features, n_bins), wide, kRowsDense);
  const BuildGeom g0 = make_geom(n_features, n_bins, n_rows, device_cu_count(), build_wg_per_cu(cap, false, wide, halves),
                                 wide, halves);
  const BuildGeom g1 = make_geom(n_features, n_bins, n_rows, device_cu_count(), build_wg_per_cu(cap, true, wide, halves),
                                 wide, halves);
  size_t b = (g0.partial_words > g1.partial_words ? g0.partial_words : g1.partial_words) * 4 +
             2 * (((size_t)n_rows + 63) / 64 * 64) * 4;  // + grad / hess of a leaf in leaf order
  // + the joint histograms of a fused copy (at most one column per feature)
  if (n_bins <= kFusedCap) b += (size_t)n_features * kFusedCap * sizeof(gbdt_bin_t);
  // gbdt_grow_tree searches the children of a round in one launch
  const size_t cand = (size_t)2 * kGrowRound * split_grouping(n_features, n_bins, 1).n_wg * sizeof(SplitCand);
  if (cand > b) b = cand;
  const size_t part = make_part_geom(n_rows > 0 ? n_rows : 1).bytes;
  if (part > b) b = part;
  return (b + 255) / 256 * 256 + kWsHeadBytes;
}

int gbdt_set_workspace(void* dev_ptr, size_t bytes) {
  if ((dev_ptr == nullptr) != (bytes == 0)) return GBDT_EINVAL;
  if (((uintptr_t)dev_ptr & 255u) != 0) return GBDT_EINVAL;
  std::lock_guard<std::mutex> lk(g_ws.mu);
  g_ws.user = dev_ptr;
  g_ws.user_bytes = bytes;
  g_ws.zeroed = g_ws.zeroed == dev_ptr ? nullptr : g_ws.zeroed;  // a caller buffer starts with unknown contents
  return GBDT_OK;
}

int gbdt_hist_build(const void* bin_matrix, int64_t n_rows, int32_t n_features, int32_t n_bins,
                    const int32_t* leaf_row_idx, int64_t n_leaf_rows, const float* grad,
                    const float* hess, gbdt_bin_t* hist_out, void* stream) {
  return hist_build_impl(bin_matrix, n_rows, n_features, n_bins, leaf_row_idx, n_leaf_rows, grad, hess, hist_out,
                         stream, nullptr, 0);
}

int gbdt_hist_build_noalloc(const void* bin_matrix, int64_t n_rows, int32_t n_features, int32_t n_bins,
                            const int32_t* leaf_row_idx, int64_t n_leaf_rows, const float* grad,
                            const float* hess, gbdt_bin_t* hist_out, void* stream) {
  void* base = nullptr;
  const int rc = noalloc_scratch_ptr(&base);
  if (rc != GBDT_OK) return rc;
  return hist_build_impl(bin_matrix, n_rows, n_features, n_bins, leaf_row_idx, n_leaf_rows, grad, hess, hist_out,
                         stream, base, kNoAllocScratchBytes);
}

size_t gbdt_hist_build_noalloc_max_partial_bytes(void) { return kNoAllocPartialBytes; }

// gbdt_hist_build_batch; with seg_off (gbdt_grow_tree: the leaves of a round are segments of its
// row buffers, not one list back to back) leaf l's rows are row_idx[seg_off[l] .. seg_off[l] + its
// length by leaf_offsets), different leaves' positions being different also modulo seg_wrap and those below n_rows; grad / hess
// read by row id are read from stat_pairs if given.
static int hist_build_batch_impl(const void* bin_matrix, int64_t n_rows, int32_t n_features,
                          int32_t n_bins, const int32_t* row_idx, const int64_t* leaf_offsets,
                          int32_t n_leaves, const float* grad, const float* hess,
                          gbdt_bin_t* hist_out, void* stream, const uint32_t* seg_off,
                          uint32_t seg_wrap = ~0u, const float2* stat_pairs = nullptr) {
  if (!valid_shape(n_rows, n_features, n_bins)) return GBDT_EINVAL;
  if (n_leaves < 0) return GBDT_EINVAL;
  if (n_leaves == 0) return GBDT_OK;
  if (!leaf_offsets || !hist_out) return GBDT_EINVAL;
  if (leaf_offsets[0] < 0) return GBDT_EINVAL;
  for (int32_t l = 0; l < n_leaves; ++l)
    if (leaf_offsets[l + 1] < leaf_offsets[l]) return GBDT_EINVAL;
  const int64_t total_rows = leaf_offsets[n_leaves] - leaf_offsets[0];
  if (total_rows > 0 && (!bin_matrix || !row_idx || !grad || !hess)) return GBDT_EINVAL;
  if (total_rows > 0 && n_rows == 0) return GBDT_EINVAL;
  if (n_rows >= ((int64_t)1 << 30)) return GBDT_EUNSUPPORTED;
  // (always from the plain tiles: the leaves of a batch are sparse in the matrix, where a fused copy's
  // wider rows cost more HBM traffic than its fewer columns save in atomics)
  const TilePlan p = make_tile_plan(n_features, n_bins);
  const int n_tiles = plan_n_tiles(p);
  if (n_tiles > 65535) return GBDT_EUNSUPPORTED;
  if ((n_rows + kEpochRows) * (int64_t)p.wm >= ((int64_t)1 << 32)) return GBDT_EUNSUPPORTED;
  const bool wide = g_wide.load() != 0;
  const bool halves = plan_halves(p, wide, rows_of_batch(total_rows, n_leaves, n_rows));
  const int cus = device_cu_count(), wg_per_cu = build_wg_per_cu(p.cap, true, wide, halves);
  const int n_parts = plan_n_parts(p, halves);
  // words of the partial blocks of one workgroup column (two blocks each with wide accumulation)
  const size_t col = (p.cap == 16 ? variant_column_words<GBDT_VARIANT_16>(p)
                                  : (p.cap == 64 ? variant_column_words<GBDT_VARIANT_64>(p)
                                                 : variant_column_words<GBDT_VARIANT_256>(p))) *
                     (wide ? 2 : 1);
  // one scratch buffer serves the launches one after the other: size it for the largest
  size_t need_words = 0;
  BatchPlan first_plan;  // (of the first launch: nearly always the only one)
  for (int32_t l0 = 0; l0 < n_leaves; l0 += kBatchLeaves) {
    const int32_t n = n_leaves - l0 < kBatchLeaves ? n_leaves - l0 : kBatchLeaves;
    for (int32_t i = 0; i < n; ++i)
      if (leaf_offsets[l0 + i + 1] - leaf_offsets[l0 + i] >= ((int64_t)1 << 31)) return GBDT_EUNSUPPORTED;
    if (leaf_offsets[l0 + n] - leaf_offsets[l0] >= ((int64_t)1 << 32)) return GBDT_EUNSUPPORTED;
    const BatchPlan b = plan_batch(leaf_offsets, l0, n, cus, wg_per_cu, n_parts, seg_off);
    if (l0 == 0) first_plan = b;
    if ((int64_t)b.total_wgs * n_parts >= ((int64_t)1 << 31)) return GBDT_EUNSUPPORTED;
    const size_t w = (size_t)b.total_wgs * col;
    if (w > need_words) need_words = w;
  }
  hipStream_t s = (hipStream_t)stream;
  if (total_rows > 0 && !seg_off) {
    const int rc_ids = check_row_ids(row_idx + leaf_offsets[0], total_rows, n_rows, s);
    if (rc_ids != GBDT_OK) return rc_ids;
  }
  // grad / hess of the whole concatenated list in list order, gathered once (see stats_gather_pays)
  // (a tree's (gradient, hessian) pairs are one line a row already)
  bool by_pos = total_rows > 0 && (stats_gather_pays(n_tiles, total_rows, total_rows / n_leaves, n_rows) ||
                                   (halves && !stat_pairs &&
                                    stats_gather_of_parts_pays(n_parts, total_rows, total_rows / n_leaves, n_rows)));
  size_t stats_words = by_pos ? 2 * (((size_t)(seg_off ? n_rows : total_rows) + 63) / 64 * 64) : 0;
  void* ws = nullptr;
  int rc = get_workspace((need_words + stats_words) * 4 + 256, s, &ws);
  if (rc == GBDT_ENOMEM && by_pos) {  // a caller's workspace sized for the partial blocks alone: no gather
    by_pos = false;
    stats_words = 0;
    rc = get_workspace(need_words * 4 + 256, s, &ws);
  }
  if (rc != GBDT_OK) return rc;
  float* g_list = (float*)ws + need_words;
  float* h_list = g_list + stats_words / 2;
  if (by_pos) {
    const bool by_parts = seg_off || (n_leaves > 1 && n_rows >= kGatherListsMinRows);
    if (!by_parts) {
      hipLaunchKernelGGL(stats_gather_kernel, dim3((unsigned)((total_rows + 255) / 256)), dim3(256), 0, s,
                         row_idx + leaf_offsets[0], grad, hess, total_rows, g_list, h_list);
      HIP_TRY(hipGetLastError());
    }
    GatherTable t;
    for (int32_t l0 = 0; by_parts && l0 < n_leaves; l0 += t.n_lists) {
      const uint32_t blocks = fill_gather_table(leaf_offsets, seg_off, l0, n_leaves, &t);
      const int64_t base = seg_off ? 0 : leaf_offsets[l0], before = seg_off ? 0 : base - leaf_offsets[0];
      if (blocks == 0) continue;
      hipLaunchKernelGGL(stats_gather_lists_kernel, dim3(blocks * kXcds), dim3(256), 0, s, row_idx + base, grad, hess, t,
                         seg_wrap, g_list + before, h_list + before);
      HIP_TRY(hipGetLastError());
    }
  }
  for (int32_t l0 = 0; l0 < n_leaves; l0 += kBatchLeaves) {
    const int32_t n = n_leaves - l0 < kBatchLeaves ? n_leaves - l0 : kBatchLeaves;
    const BatchPlan b = l0 == 0 ? first_plan : plan_batch(leaf_offsets, l0, n, cus, wg_per_cu, n_parts, seg_off);
    BatchMergeArgs m;
    m.m.partials = (const uint32_t*)ws;
    m.m.out = hist_out + (size_t)l0 * n_features * n_bins;
    m.m.plan = p;
    m.m.n_features = n_features;
    m.m.n_bins = n_bins;
    m.m.chunks_main = 0;
    m.m.chunks_rem = 0;
    m.m.halves = halves ? 1 : 0;
    m.m.counters = nullptr;
    m.column_words = col;
    m.blocks_per_wg = wide ? 2 : 1;
    // the leaves the pass has work for: empty ones (zeros) and those of several workgroups per tile
    int n_merge = 0;
    for (int32_t i = 0; i < n; ++i)
      if (batch_wgs(b.leaf[i]) != 1u) m.leaf[n_merge++] = b.leaf[i];
    if (b.total_wgs > 0) {
      BatchArgs a;
      a.packed = (const uint8_t*)bin_matrix;
      a.idx = seg_off ? row_idx : row_idx + leaf_offsets[l0];
      const int64_t stats_at = seg_off ? 0 : leaf_offsets[l0] - leaf_offsets[0];
      a.grad = by_pos ? g_list + stats_at : grad;
      a.hess = by_pos ? h_list + stats_at : hess;
      a.stat_wrap = seg_wrap;
      a.stats_by_pos = by_pos ? 1 : 0;
      a.stat_shift = 2;
      if (stat_pairs && !by_pos) {
        a.grad = (const float*)stat_pairs;
        a.hess = (const float*)stat_pairs + 1;
        a.stat_shift = 3;
      }
      a.partials = (uint32_t*)ws;
      a.n_rows = n_rows;
      a.n_main = p.n_main;
      a.wr = p.wr;
      a.line_tiles = plan_line_tiles(n_rows);
      a.deal = deal_order(a.line_tiles, b.most_unit_epochs, (int64_t)b.total_wgs * n_parts, cus, wide);
      a.n_leaves = n;
      a.n_cols = b.total_wgs;
      a.hist_out = hist_out + (size_t)l0 * n_features * n_bins;
      a.n_features = n_features;
      a.n_bins = n_bins;
      memcpy(a.leaf, b.leaf, sizeof a.leaf);
      const int blocks = (int)b.total_wgs * n_parts;
      const bool is_short = batch_is_short(b, p.cap, wide);
      if (wide) {
        if (p.cap == 16) {
          rc = launch_build_batch<GBDT_VARIANT_16W, true>(a, blocks, s, is_short);
        } else if (p.cap == 64) {
          rc = launch_build_batch<GBDT_VARIANT_64W, true>(a, blocks, s, is_short);
        } else if (halves) {
          rc = launch_build_batch<GBDT_VARIANT_256W_HALVES, true, true>(a, blocks, s, is_short);
        } else {
          rc = launch_build_batch<GBDT_VARIANT_256W, true>(a, blocks, s, is_short);
        }
      } else if (p.cap == 16) {
        rc = launch_build_batch<GBDT_VARIANT_16>(a, blocks, s, is_short);
      } else if (p.cap == 64) {
        rc = launch_build_batch<GBDT_VARIANT_64>(a, blocks, s, is_short);
      } else {
        rc = launch_build_batch<GBDT_VARIANT_256>(a, blocks, s, is_short);
      }
      if (rc != GBDT_OK) return rc;
    }
    if (n_merge == 0) continue;
    const int64_t tile_cells = merge_tile_cells(p, n_bins);
    int32_t most_chunks = 0;
    for (int i = 0; i < n_merge; ++i) {
      const int32_t c = (int32_t)batch_wgs(m.leaf[i]) * (wide ? 2 : 1);
      most_chunks = c > most_chunks ? c : most_chunks;
    }
    const int parts = merge_parts(tile_cells, (int64_t)n_tiles * n_merge, most_chunks);
    const dim3 merge_grid((unsigned)((tile_cells + merge_wg_cells(parts) - 1) / merge_wg_cells(parts)), n_tiles, n_merge);
    auto merge = [&](auto kernel) { hipLaunchKernelGGL(kernel, merge_grid, dim3(merge_wg_threads(parts)), 0, s, m); };
    merge(parts == 1 ? hist_merge_batch_kernel<1> : parts == 2 ? hist_merge_batch_kernel<2>
          : parts == 4 ? hist_merge_batch_kernel<4>
          : parts == kMergePartsMost ? hist_merge_batch_kernel<kMergePartsMost> : hist_merge_batch_kernel<kMergePartsWide>);
    HIP_TRY(hipGetLastError());
  }
  return GBDT_OK;
}

int gbdt_hist_build_batch(const void* bin_matrix, int64_t n_rows, int32_t n_features,
                          int32_t n_bins, const int32_t* row_idx, const int64_t* leaf_offsets,
                          int32_t n_leaves, const float* grad, const float* hess,
                          gbdt_bin_t* hist_out, void* stream) {
  return hist_build_batch_impl(bin_matrix, n_rows, n_features, n_bins, row_idx, leaf_offsets, n_leaves, grad, hess,
                               hist_out, stream, nullptr);
}

size_t gbdt_hist_build_batch_workspace_bytes(int32_t n_features, int32_t n_bins, int32_t n_leaves) {
  if (n_features <= 0 || n_bins < 2 || n_bins > 256 || n_leaves < 0) return 0;
  const TilePlan p = make_tile_plan(n_features, n_bins);
  const bool wide = g_wide.load() != 0;
  const bool halves = plan_halves(p, wide, kRowsSparse);  // (a call that takes whole tiles has fewer columns)
  const int n_parts = plan_n_parts(p, halves);
  const int64_t resident = (int64_t)device_cu_count() * build_wg_per_cu(p.cap, true, wide, halves);
  const size_t col = (p.cap == 16 ? variant_column_words<GBDT_VARIANT_16>(p)
                                  : (p.cap == 64 ? variant_column_words<GBDT_VARIANT_64>(p)
                                                 : variant_column_words<GBDT_VARIANT_256>(p))) *
                     (wide ? 2 : 1);
  // the leaves of a launch share the resident workgroups, and each has at least one per tile: plan_batch takes
  // no plan of more columns than that
  int64_t budget = resident / n_parts;
  if (budget < 1) budget = 1;
  const int64_t per_launch = n_leaves < kBatchLeaves ? n_leaves : kBatchLeaves;
  // (the call gathers grad / hess into list order only when the scratch has 8 more bytes per listed
  // row to spare; with a caller buffer of exactly this size it reads them by row id)
  const size_t b = (size_t)(budget + per_launch) * col * 4 + 256;
  return (b + 255) / 256 * 256 + kWsHeadBytes;
}

int gbdt_hist_subtract(const gbdt_bin_t* parent, const gbdt_bin_t* child, gbdt_bin_t* sibling_out,
                       int32_t n_features, int32_t n_bins, void* stream) {
  if (!parent || !child || !sibling_out) return GBDT_EINVAL;
  if (n_features <= 0 || n_bins < 2 || n_bins > 256) return GBDT_EINVAL;
  const int32_t n = n_features * n_bins;
  hipLaunchKernelGGL(hist_subtract_kernel, dim3((n + 255) / 256), dim3(256), 0,
                     (hipStream_t)stream, parent, child, sibling_out, n);
  HIP_TRY(hipGetLastError());
  return GBDT_OK;
}

int gbdt_best_split_batch(const gbdt_bin_t* hists, int32_t n_hists, float lambda,
                          float min_child_hess, gbdt_split_t* splits_out, int32_t n_features,
                          int32_t n_bins, void* stream) {
  if (n_hists < 0) return GBDT_EINVAL;
  if (n_features <= 0 || n_bins < 2 || n_bins > 256) return GBDT_EINVAL;
  if (!(lambda >= 0.0f)) return GBDT_EINVAL;
  if (n_hists == 0) return GBDT_OK;
  if (!hists || !splits_out) return GBDT_EINVAL;
  const int64_t stride = (int64_t)n_features * n_bins;
  for (int32_t h0 = 0; h0 < n_hists; h0 += kSplitMaxHists) {
    const int32_t nh = n_hists - h0 < kSplitMaxHists ? n_hists - h0 : kSplitMaxHists;
    const int rc = launch_split(hists + (size_t)h0 * stride, stride, nh, lambda, min_child_hess,
                                splits_out + h0, n_features, n_bins, (hipStream_t)stream);
    if (rc != GBDT_OK) return rc;
  }
  return GBDT_OK;
}

int gbdt_best_split(const gbdt_bin_t* hist, float lambda, float min_child_hess,
                    gbdt_split_t* split_out, int32_t n_features, int32_t n_bins, void* stream) {
  if (!hist || !split_out) return GBDT_EINVAL;
  return gbdt_best_split_batch(hist, 1, lambda, min_child_hess, split_out, n_features, n_bins,
                               stream);
}

int gbdt_partition_rows(const void* bin_matrix, int64_t n_rows, int32_t n_features,
                        int32_t n_bins, const int32_t* leaf_row_idx, int64_t n_leaf_rows,
                        const gbdt_split_t* split, int32_t* children_out, int64_t* n_left_out,
                        void* stream) {
  if (!valid_shape(n_rows, n_features, n_bins)) return GBDT_EINVAL;
  if (!bin_matrix || !split || !children_out) return GBDT_EINVAL;
  if (n_leaf_rows < 0) return GBDT_EINVAL;
  if (!leaf_row_idx && n_leaf_rows > n_rows) return GBDT_EINVAL;
  if (n_rows == 0 && n_leaf_rows > 0) return GBDT_EINVAL;
  if (n_rows >= ((int64_t)1 << 30) || n_leaf_rows >= ((int64_t)1 << 31)) return GBDT_EUNSUPPORTED;
  hipStream_t s = (hipStream_t)stream;
  {
    const int rc_ids = check_row_ids(leaf_row_idx, n_leaf_rows, n_rows, s);
    if (rc_ids != GBDT_OK) return rc_ids;
  }
  const TilePlan p = make_tile_plan(n_features, n_bins);
  if (n_leaf_rows <= (int64_t)kPartThreads * kPartOneSteps) {  // small leaf: one workgroup, one launch
    hipLaunchKernelGGL(partition_one_kernel, dim3(1), dim3(kPartThreads), 0, s, (const uint8_t*)bin_matrix,
                       n_rows, n_features, p, leaf_row_idx, (int32_t)n_leaf_rows, split, children_out,
                       n_left_out);
    HIP_TRY(hipGetLastError());
    return GBDT_OK;
  }
  const PartGeom g = make_part_geom(n_leaf_rows > 0 ? n_leaf_rows : 1);
  void* ws = nullptr;
  int rc = get_workspace(g.bytes, s, &ws);
  if (rc != GBDT_OK) return rc;
  uint64_t* flags = (uint64_t*)ws;
  uint32_t* chunk_left = (uint32_t*)(flags + g.flag_words);
  hipLaunchKernelGGL(partition_flag_kernel, dim3(g.n_chunks), dim3(kPartThreads), 0, s,
                     (const uint8_t*)bin_matrix, n_rows, n_features, p, leaf_row_idx, n_leaf_rows,
                     split, g.rows_per_thread, flags, chunk_left);
  HIP_TRY(hipGetLastError());
  hipLaunchKernelGGL(partition_scatter_kernel, dim3(g.n_chunks), dim3(kPartThreads), 0, s,
                     leaf_row_idx, n_leaf_rows, g.rows_per_thread, (const uint64_t*)flags,
                     (const uint32_t*)chunk_left, g.n_chunks, children_out, n_left_out);
  HIP_TRY(hipGetLastError());
  return GBDT_OK;
}

// gbdt_partition_rows_batch; with split_idx (gbdt_grow_tree_depthwise) leaf l's record is splits[split_idx[l]], kNoSplitRecord
// for none, and a lone leaf of all rows may come without a list.
static int partition_rows_batch_impl(const void* bin_matrix, int64_t n_rows, int32_t n_features,
                                     int32_t n_bins, const int32_t* row_idx, const int64_t* leaf_offsets,
                                     int32_t n_leaves, const gbdt_split_t* splits, const uint32_t* split_idx,
                                     int32_t* children_out, int64_t* n_left_out, void* stream) {
  if (!valid_shape(n_rows, n_features, n_bins)) return GBDT_EINVAL;
  if (n_leaves < 0) return GBDT_EINVAL;
  if (n_leaves == 0) return GBDT_OK;
  if (!leaf_offsets || !splits) return GBDT_EINVAL;
  if (leaf_offsets[0] < 0) return GBDT_EINVAL;
  int64_t longest = 0;
  for (int32_t l = 0; l < n_leaves; ++l) {
    const int64_t n = leaf_offsets[l + 1] - leaf_offsets[l];
    if (n < 0) return GBDT_EINVAL;
    if (n >= ((int64_t)1 << 31)) return GBDT_EUNSUPPORTED;
    if (n > longest) longest = n;
  }
  const int64_t total_rows = leaf_offsets[n_leaves] - leaf_offsets[0];
  if (total_rows > 0 && (!bin_matrix || (!row_idx && !split_idx) || !children_out)) return GBDT_EINVAL;
  if (total_rows > 0 && n_rows == 0) return GBDT_EINVAL;
  if (n_rows >= ((int64_t)1 << 30)) return GBDT_EUNSUPPORTED;
  hipStream_t s = (hipStream_t)stream;
  if (total_rows > 0 && !split_idx) {
    const int rc_ids = check_row_ids(row_idx + leaf_offsets[0], total_rows, n_rows, s);
    if (rc_ids != GBDT_OK) return rc_ids;
  }
  // chunks of 256 * rows_per_thread positions, at most kPartMaxChunks per leaf
  const int32_t rpt = make_part_geom(longest > 0 ? longest : 1).rows_per_thread;
  const int64_t chunk_rows = (int64_t)kPartThreads * rpt;
  // scratch for the launch with the most chunks
  int64_t max_chunks = 0;
  for (int32_t l0 = 0; l0 < n_leaves; l0 += kPartBatchLeaves) {
    const int32_t n = n_leaves - l0 < kPartBatchLeaves ? n_leaves - l0 : kPartBatchLeaves;
    if (leaf_offsets[l0 + n] - leaf_offsets[l0] >= ((int64_t)1 << 32)) return GBDT_EUNSUPPORTED;
    int64_t chunks = 0;
    for (int32_t i = 0; i < n; ++i)
      chunks += (leaf_offsets[l0 + i + 1] - leaf_offsets[l0 + i] + chunk_rows - 1) / chunk_rows;
    if (chunks > max_chunks) max_chunks = chunks;
  }
  if (max_chunks >= ((int64_t)1 << 31)) return GBDT_EUNSUPPORTED;
  const size_t flag_words = (size_t)max_chunks * rpt * kPartWaves;
  void* ws = nullptr;
  int rc = get_workspace(flag_words * 8 + (size_t)max_chunks * 4 + 256, s, &ws);
  if (rc != GBDT_OK) return rc;
  const TilePlan p = make_tile_plan(n_features, n_bins);
  for (int32_t l0 = 0; l0 < n_leaves; l0 += kPartBatchLeaves) {
    const int32_t n = n_leaves - l0 < kPartBatchLeaves ? n_leaves - l0 : kPartBatchLeaves;
    PartBatchArgs a;
    a.packed = (const uint8_t*)bin_matrix;
    a.idx = row_idx ? row_idx + leaf_offsets[l0] : nullptr;
    a.split = split_idx ? splits : splits + l0;
    a.out = children_out + leaf_offsets[l0];
    a.n_left_out = n_left_out ? n_left_out + l0 : nullptr;
    a.flags = (uint64_t*)ws;
    a.chunk_left = (uint32_t*)(a.flags + flag_words);
    a.n_rows = n_rows;
    a.plan = p;
    a.n_features = n_features;
    a.rows_per_thread = rpt;
    a.n_leaves = n;
    uint32_t chunks = 0;
    bool any_empty = false;
    for (int32_t i = 0; i < kPartBatchLeaves; ++i) {
      PartLeaf& lf = a.leaf[i];
      if (i < n) {
        lf.row_off = lf.out_off = (uint32_t)(leaf_offsets[l0 + i] - leaf_offsets[l0]);
        lf.n = (uint32_t)(leaf_offsets[l0 + i + 1] - leaf_offsets[l0 + i]);
        lf.split_idx = split_idx ? split_idx[l0 + i] : (uint32_t)i;
        lf.first_chunk = chunks;
        chunks += (uint32_t)(((int64_t)lf.n + chunk_rows - 1) / chunk_rows);
        any_empty = any_empty || lf.n == 0;
      } else {
        lf.row_off = lf.out_off = lf.n = lf.split_idx = 0;
        lf.first_chunk = chunks;
      }
    }
    a.n_chunks = chunks;
    if (n_left_out && any_empty) {
      hipLaunchKernelGGL(partition_empty_counts_kernel, dim3((n + 255) / 256), dim3(256), 0, s, a);
      HIP_TRY(hipGetLastError());
    }
    if (chunks == 0) continue;
    hipLaunchKernelGGL(partition_flag_batch_kernel, dim3(chunks), dim3(kPartThreads), 0, s, a);
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(partition_scatter_batch_kernel, dim3(chunks), dim3(kPartThreads), 0, s, a);
    HIP_TRY(hipGetLastError());
  }
  return GBDT_OK;
}

int gbdt_partition_rows_batch(const void* bin_matrix, int64_t n_rows, int32_t n_features,
                              int32_t n_bins, const int32_t* row_idx, const int64_t* leaf_offsets,
                              int32_t n_leaves, const gbdt_split_t* splits, int32_t* children_out,
                              int64_t* n_left_out, void* stream) {
  return partition_rows_batch_impl(bin_matrix, n_rows, n_features, n_bins, row_idx, leaf_offsets, n_leaves, splits, nullptr,
                                   children_out, n_left_out, stream);
}

// --- leaf-wise tree growth -------------------------------------------------------------

size_t gbdt_grow_tree_scratch_bytes(int64_t n_rows, int32_t n_features, int32_t n_bins,
                                    int32_t max_leaves) {
  if (!valid_shape(n_rows, n_features, n_bins) || max_leaves < 1) return 0;
  return tree_scratch_layout(n_rows, n_features, n_bins, max_leaves).total;
}

int gbdt_grow_tree(const void* bin_matrix, int64_t n_rows, int32_t n_features, int32_t n_bins,
                   const float* grad, const float* hess, int32_t max_leaves, float lambda,
                   float min_child_hess, float min_split_gain, void* scratch, size_t scratch_bytes,
                   gbdt_tree_node_t* nodes_out, int32_t* n_nodes_out, int32_t* row_order_out,
                   void* stream) {
  if (!valid_shape(n_rows, n_features, n_bins)) return GBDT_EINVAL;
  if (max_leaves < 1 || !nodes_out || !n_nodes_out || !scratch) return GBDT_EINVAL;
  if (!(lambda >= 0.0f) || min_split_gain != min_split_gain) return GBDT_EINVAL;
  if (n_rows > 0 && (!bin_matrix || !grad || !hess)) return GBDT_EINVAL;
  if (((uintptr_t)scratch & 255u) != 0) return GBDT_EINVAL;
  if (n_rows >= ((int64_t)1 << 30)) return GBDT_EUNSUPPORTED;
  const TreeScratch lay = tree_scratch_layout(n_rows, n_features, n_bins, max_leaves);
  if (scratch_bytes < lay.least) return GBDT_ENOMEM;
  HostRecords found(2 * kGrowRound);  // the records of the last search
  if (!found.ok()) {
    snprintf(g_hip_err, sizeof g_hip_err, "no page-locked host memory for the split records");
    return GBDT_ENOMEM;
  }
  hipStream_t s = (hipStream_t)stream;
  char* base = (char*)scratch;
  int32_t* rows_base = (int32_t*)(base + lay.rows_a);   // row buffer b starts b * row_elems entries in
  gbdt_bin_t* pool = (gbdt_bin_t*)(base + lay.hists);
  gbdt_split_t* recs = (gbdt_split_t*)(base + lay.recs);            // record of the histogram in slot i
  const size_t hist_elems = (size_t)n_features * n_bins;
  const TilePlan plan = make_tile_plan(n_features, n_bins);

  // Best-first growth is sequential by definition: the open leaf with the largest gain is split,
  // its children join the open leaves, and so on (the older leaf on equal gains).  To wait for
  // the device once per ROUND instead of once per split, a round expands (partitions, builds,
  // searches) the best few open leaves at once; the host then replays the sequential rule on
  // what it knows and stops at the first leaf whose children it has not seen yet.  Every node
  // the replay splits is one the sequential rule splits, in the same order, so the tree is the
  // sequential one; an expansion the replay never reaches before the leaf budget is used up is
  // dropped (its leaf keeps its rows: children are written to the other row buffer).
  struct Cand {            // a node whose histogram exists on the device
    int64_t begin;         // its rows: positions [begin, begin + count) of row buffer `buf`
    uint32_t count;
    int buf;
    int slot;              // histogram slot in the pool
    gbdt_split_t rec;      // its best split
    float sum_grad, sum_hess;
    int kid[2];            // children once expanded (-1: not yet)
    int id;                // node id once it belongs to the tree
  };
  std::vector<Cand> cands;
  cands.reserve(1 + 2 * (size_t)grow_max_expansions(max_leaves));
  auto fill_node = [&](int k, int parent, const Cand& c) {
    gbdt_tree_node_t& nd = nodes_out[k];
    nd.parent = parent;
    nd.left = nd.right = -1;
    nd.feature = c.rec.feature;
    nd.bin = c.rec.bin;
    nd.gain = c.rec.gain;
    nd.sum_grad = c.sum_grad;
    nd.sum_hess = c.sum_hess;
    nd.count = c.count;
    nd.reserved = 0;
    nd.row_begin = c.begin;
  };

  // root: histogram and first partition without an index list
  int rc = gbdt_hist_build(bin_matrix, n_rows, n_features, n_bins, nullptr, n_rows, grad, hess, pool, s);
  if (rc != GBDT_OK) return rc;
  rc = found.enqueued(launch_split(pool, 0, 1, lambda, min_child_hess, recs, n_features, n_bins, s, found.device()));
  if (rc != GBDT_OK) return rc;
  const float2* stat_pairs = nullptr;
  if (lay.total > lay.least && scratch_bytes >= lay.total && max_leaves > 1) {
    float2* pairs = (float2*)(base + lay.pairs);
    hipLaunchKernelGGL(stats_pair_kernel, dim3(device_cu_count() * 8), dim3(256), 0, s, grad, hess, n_rows, pairs);
    HIP_TRY(hipGetLastError());
    stat_pairs = pairs;
  }
  HIP_TRY(found.wait(s));
  {
    Cand root;
    root.begin = 0;
    root.count = (uint32_t)n_rows;
    root.buf = 0;
    root.slot = 0;
    root.rec = found[0];
    if (!split_fits(root.rec, root.count)) return GBDT_EHIP;
    root.kid[0] = root.kid[1] = -1;
    root.id = 0;
    root.sum_grad = root.rec.left_grad + root.rec.right_grad;
    root.sum_hess = root.rec.left_hess + root.rec.right_hess;
    if (root.rec.feature < 0 && n_rows > 0) {
      // no split record carries the totals: sum feature 0's bins on the host
      std::vector<gbdt_bin_t> row((size_t)n_bins);
      HIP_TRY(hipMemcpyAsync(row.data(), pool, (size_t)n_bins * sizeof(gbdt_bin_t), hipMemcpyDeviceToHost, s));
      HIP_TRY(hipStreamSynchronize(s));
      double g = 0.0, h = 0.0;
      for (const gbdt_bin_t& b : row) {
        g += b.grad;
        h += b.hess;
      }
      root.sum_grad = (float)g;
      root.sum_hess = (float)h;
    }
    cands.push_back(root);
    fill_node(0, -1, root);
  }
  auto eligible = [&](const Cand& c) { return c.rec.feature >= 0 && c.rec.gain > min_split_gain; };
  std::vector<int> open = {0};  // candidates that are leaves of the tree so far
  int n_nodes = 1, n_leaves = 1, next_slot = 1;
  int expansions = 0, splits = 0, rounds = 0;
  const int spec_budget = grow_speculative_budget(max_leaves);
  // (host clock, for the trace line: all rounds, and the part of them spent waiting for the stream)
  double wait_us = 0, rounds_us = 0;
  auto last_round_end = std::chrono::steady_clock::now();
  for (;;) {
    // ---- replay the sequential rule as far as the expansions seen so far carry it
    int blocked = -1;
    while (n_leaves < max_leaves) {
      int m = -1;
      for (int h : open) {  // larger gain, then smaller node id
        const Cand& c = cands[h];
        if (!eligible(c)) continue;
        if (m < 0 || c.rec.gain > cands[m].rec.gain || (c.rec.gain == cands[m].rec.gain && c.id < cands[m].id)) m = h;
      }
      if (m < 0) break;
      if (cands[m].kid[0] < 0) {
        blocked = m;
        break;
      }
      const int left = n_nodes, right = n_nodes + 1;
      nodes_out[cands[m].id].left = left;
      nodes_out[cands[m].id].right = right;
      for (int side = 0; side < 2; ++side) {
        Cand& k = cands[cands[m].kid[side]];
        k.id = side == 0 ? left : right;
        fill_node(k.id, cands[m].id, k);
        open.push_back(cands[m].kid[side]);
      }
      open.erase(std::find(open.begin(), open.end(), m));
      n_nodes += 2;
      n_leaves += 1;
      splits += 1;
    }
    if (blocked < 0) break;  // leaf budget used up, or nothing left to split
    // ---- this round: the blocking leaf and the next best open leaves without children
    // (A width that follows the number of splits the last round made possible was tried: fewer
    // leaves expanded in vain on deep, chain-like trees, but more rounds, and rounds cost more.)
    int extra = kGrowRound - 1;
    if (extra > max_leaves - n_leaves - 1) extra = max_leaves - n_leaves - 1;
    if (extra > spec_budget - (expansions - splits)) extra = spec_budget - (expansions - splits);
    if (extra < 0) extra = 0;
    std::vector<int> batch = {blocked};
    if (extra > 0) {
      std::vector<int> more;
      for (int h : open)
        if (h != blocked && cands[h].kid[0] < 0 && eligible(cands[h])) more.push_back(h);
      std::sort(more.begin(), more.end(), [&](int x, int y) {
        return cands[x].rec.gain > cands[y].rec.gain || (cands[x].rec.gain == cands[y].rec.gain && cands[x].id < cands[y].id);
      });
      if ((int)more.size() > extra) more.resize(extra);
      batch.insert(batch.end(), more.begin(), more.end());
    }
    const int k = (int)batch.size();
    if (next_slot + 2 * k > lay.n_slots) return GBDT_ENOMEM;  // (cannot happen: the budget above bounds it)

    // ---- partition the k leaves: children into the other row buffer, same positions; every leaf's
    // split record is read on the device, from the records by histogram slot
    {
      uint32_t longest = 1;
      for (int j = 0; j < k; ++j) longest = cands[batch[j]].count > longest ? cands[batch[j]].count : longest;
      const int32_t rpt = make_part_geom(longest).rows_per_thread;
      const int64_t chunk_rows = (int64_t)kPartThreads * rpt;
      PartBatchArgs a;
      a.packed = (const uint8_t*)bin_matrix;
      a.idx = rounds == 0 ? nullptr : rows_base;  // (the root's rows are 0, 1, 2, ...: no list)
      a.split = recs;
      a.out = rows_base;
      a.n_left_out = nullptr;
      a.n_rows = n_rows;
      a.plan = plan;
      a.n_features = n_features;
      a.rows_per_thread = rpt;
      a.n_leaves = k;
      uint32_t chunks = 0;
      for (int j = 0; j < kPartBatchLeaves; ++j) {
        PartLeaf& lf = a.leaf[j];
        lf.row_off = lf.out_off = lf.n = lf.split_idx = 0;
        lf.first_chunk = chunks;
        if (j < k) {
          const Cand& c = cands[batch[j]];
          lf.row_off = (uint32_t)(c.begin + (int64_t)c.buf * (int64_t)lay.row_elems);
          lf.out_off = (uint32_t)(c.begin + (int64_t)(1 - c.buf) * (int64_t)lay.row_elems);
          lf.n = c.count;
          lf.split_idx = (uint32_t)c.slot;
          chunks += (uint32_t)(((int64_t)lf.n + chunk_rows - 1) / chunk_rows);
        }
      }
      a.n_chunks = chunks;
      const size_t flag_words = (size_t)chunks * rpt * kPartWaves;
      void* ws = nullptr;
      rc = get_workspace(flag_words * 8 + (size_t)chunks * 4 + 256, s, &ws);
      if (rc != GBDT_OK) return rc;
      a.flags = (uint64_t*)ws;
      a.chunk_left = (uint32_t*)(a.flags + flag_words);
      if (chunks > 0) {
        hipLaunchKernelGGL(partition_flag_batch_kernel, dim3(chunks), dim3(kPartThreads), 0, s, a);
        HIP_TRY(hipGetLastError());
        hipLaunchKernelGGL(partition_scatter_batch_kernel, dim3(chunks), dim3(kPartThreads), 0, s, a);
        HIP_TRY(hipGetLastError());
      }
    }
    // ---- the smaller children's histograms in one batched build, straight from their segments of the row buffers
    std::vector<int64_t> small_offs = {0};
    std::vector<uint32_t> small_seg((size_t)k);
    std::vector<int> left_small((size_t)k);
    for (int j = 0; j < k; ++j) {
      const Cand& c = cands[batch[j]];
      const uint32_t nl = c.rec.left_count, nr = c.rec.right_count;
      left_small[j] = nl <= nr;
      const int64_t kid_base = c.begin + (int64_t)(1 - c.buf) * (int64_t)lay.row_elems;
      small_seg[j] = (uint32_t)(left_small[j] ? kid_base : kid_base + nl);
      small_offs.push_back(small_offs.back() + (left_small[j] ? nl : nr));
    }
    gbdt_bin_t* h_small = pool + (size_t)next_slot * hist_elems;  // k slots: the built children; then k: their siblings
    rc = hist_build_batch_impl(bin_matrix, n_rows, n_features, n_bins, rows_base, small_offs.data(), k, grad,
                               hess, h_small, s, small_seg.data(), (uint32_t)lay.row_elems, stat_pairs);
    if (rc != GBDT_OK) return rc;
    // ---- best splits of the 2k children, one launch, which first forms the k siblings as parent -
    // built child; the records also land in `found`
    {
      SplitSiblings sib;
      sib.pool = pool;
      sib.first = k;
      sib.n = k;
      sib.keep = 1;
      for (int j = 0; j < kSplitSiblings; ++j) sib.parent_slot[j] = j < k ? cands[batch[j]].slot : 0;
      rc = found.enqueued(launch_split(h_small, (int64_t)hist_elems, 2 * k, lambda, min_child_hess, recs + next_slot, n_features,
                                       n_bins, s, found.device(), &sib));
      if (rc != GBDT_OK) return rc;
    }
    {
      auto t0 = std::chrono::steady_clock::now();
      HIP_TRY(found.wait(s));
      auto t1 = std::chrono::steady_clock::now();
      wait_us += std::chrono::duration<double, std::micro>(t1 - t0).count();
      rounds_us += std::chrono::duration<double, std::micro>(t1 - last_round_end).count();
      last_round_end = t1;
    }
    for (int j = 0; j < k; ++j) {
      const int par = batch[j];
      const Cand pc = cands[par];
      const uint32_t nl = pc.rec.left_count, nr = pc.rec.right_count;
      for (int side = 0; side < 2; ++side) {
        const bool is_small = (side == 0) == (left_small[j] != 0);
        Cand c;
        c.begin = side == 0 ? pc.begin : pc.begin + nl;
        c.count = side == 0 ? nl : nr;
        c.buf = 1 - pc.buf;
        c.slot = is_small ? next_slot + j : next_slot + k + j;
        c.rec = found[is_small ? j : k + j];
        if (!split_fits(c.rec, c.count)) return GBDT_EHIP;
        c.sum_grad = side == 0 ? pc.rec.left_grad : pc.rec.right_grad;
        c.sum_hess = side == 0 ? pc.rec.left_hess : pc.rec.right_hess;
        c.kid[0] = c.kid[1] = -1;
        c.id = -1;
        cands[par].kid[side] = (int)cands.size();
        cands.push_back(c);
      }
    }
    next_slot += 2 * k;
    expansions += k;
    rounds += 1;
  }
  *n_nodes_out = n_nodes;
  {
    static const bool trace = [] {
      const char* e = getenv("GBDT_HIST_TRACE_TREE");  // tuning aid: one line per tree on stderr
      return e && atoi(e) > 0;
    }();
    if (trace)
      fprintf(stderr, "gbdt_grow_tree: %d leaves, %d rounds, %d leaves expanded, %d of them never split; rounds %.0f us, "
              "of which %.0f us waiting for the stream\n", n_leaves,
              rounds, expansions, expansions - splits, rounds_us, wait_us);
  }
  if (row_order_out && n_rows > 0) {
    if (n_nodes == 1) {  // never split: the rows in their own order
      hipLaunchKernelGGL(row_iota_kernel, dim3((unsigned)((n_rows + 255) / 256)), dim3(256), 0, s,
                         row_order_out, n_rows);
      HIP_TRY(hipGetLastError());
    } else {
      // the leaves' segments in position order, a table-full per launch
      std::vector<std::pair<uint32_t, int>> segs;  // (begin, buffer)
      for (int h : open) segs.emplace_back((uint32_t)cands[h].begin, cands[h].buf);
      std::sort(segs.begin(), segs.end());
      for (size_t s0 = 0; s0 < segs.size(); s0 += kSegTable) {
        SegTable t;
        const size_t ns = segs.size() - s0 < (size_t)kSegTable ? segs.size() - s0 : (size_t)kSegTable;
        for (size_t j = 0; j < ns; ++j)
          t.start[j] = segs[s0 + j].first | ((uint32_t)segs[s0 + j].second << 31);
        t.n_seg = (int32_t)ns;
        t.end = s0 + ns < segs.size() ? segs[s0 + ns].first : (uint32_t)n_rows;
        const uint32_t span = t.end - segs[s0].first;
        hipLaunchKernelGGL(leaf_rows_gather_kernel, dim3((span + kSegRows - 1) / kSegRows), dim3(256), 0,
                           s, (const int32_t*)rows_base, (const int32_t*)(rows_base + lay.row_elems), t,
                           row_order_out);
        HIP_TRY(hipGetLastError());
      }
    }
  }
  return GBDT_OK;
}

// --- level-wise tree growth ------------------------------------------------------------

size_t gbdt_grow_tree_depthwise_scratch_bytes(int64_t n_rows, int32_t n_features, int32_t n_bins,
                                              int32_t max_depth) {
  if (!valid_shape(n_rows, n_features, n_bins) || max_depth < 0 || max_depth > kMaxTreeDepth) return 0;
  return level_scratch_layout(n_rows, n_features, n_bins, max_depth).total;
}

int gbdt_grow_tree_depthwise(const void* bin_matrix, int64_t n_rows, int32_t n_features,
                             int32_t n_bins, const float* grad, const float* hess, int32_t max_depth,
                             float lambda, float min_child_hess, float min_split_gain, void* scratch,
                             size_t scratch_bytes, gbdt_tree_node_t* nodes_out, int32_t* n_nodes_out,
                             int32_t* row_order_out, void* stream) {
  if (!valid_shape(n_rows, n_features, n_bins)) return GBDT_EINVAL;
  if (max_depth < 0 || max_depth > kMaxTreeDepth || !nodes_out || !n_nodes_out || !scratch) return GBDT_EINVAL;
  if (!(lambda >= 0.0f) || min_split_gain != min_split_gain) return GBDT_EINVAL;
  if (n_rows > 0 && (!bin_matrix || !grad || !hess)) return GBDT_EINVAL;
  if (((uintptr_t)scratch & 255u) != 0) return GBDT_EINVAL;
  if (n_rows >= ((int64_t)1 << 30)) return GBDT_EUNSUPPORTED;
  const LevelScratch lay = level_scratch_layout(n_rows, n_features, n_bins, max_depth);
  if (scratch_bytes < lay.total) return GBDT_ENOMEM;
  const size_t width = (size_t)1 << max_depth;  // most nodes a level can hold
  HostRecords found(width);  // the records of the last search
  if (!found.ok()) {
    snprintf(g_hip_err, sizeof g_hip_err, "no page-locked host memory for the split records");
    return GBDT_ENOMEM;
  }
  hipStream_t s = (hipStream_t)stream;
  char* base = (char*)scratch;
  int32_t* rows_buf[2] = {(int32_t*)(base + lay.rows_a), (int32_t*)(base + lay.rows_b)};
  gbdt_bin_t* hist_buf[2] = {(gbdt_bin_t*)(base + lay.hists_a), (gbdt_bin_t*)(base + lay.hists_b)};
  gbdt_split_t* recs = (gbdt_split_t*)(base + lay.recs);
  const size_t hist_elems = (size_t)n_features * n_bins;

  auto fill_node = [&](int k, int parent, const gbdt_split_t& r, float sg, float sh, uint32_t cnt,
                       int64_t begin) {
    gbdt_tree_node_t& nd = nodes_out[k];
    nd.parent = parent;
    nd.left = nd.right = -1;
    nd.feature = r.feature;
    nd.bin = r.bin;
    nd.gain = r.gain;
    nd.sum_grad = sg;
    nd.sum_hess = sh;
    nd.count = cnt;
    nd.reserved = 0;
    nd.row_begin = begin;
  };

  // root: its histogram, and the first partition, without an index list
  int cur = 0;  // row buffer and histogram buffer of the current level
  int rc = gbdt_hist_build(bin_matrix, n_rows, n_features, n_bins, nullptr, n_rows, grad, hess, hist_buf[cur], s);
  if (rc != GBDT_OK) return rc;
  int32_t* rows_now = nullptr;  // the rows of the current level (NULL: 0, 1, 2, ...)
  // the level: its nodes in position order with their histogram slots; `frontier` also holds
  // the finished leaves, whose rows every later partition copies through unchanged
  struct Entry {
    int node;   // node id
    int slot;   // histogram slot in hist_buf[cur]; -1: a finished leaf
  };
  std::vector<Entry> frontier = {{0, 0}};
  int n_nodes = 1;
  bool root_done = false;
  SplitSiblings level_sib;  // the level's siblings, where the split search forms them
  level_sib.n = 0;
  for (int depth = 0;; ++depth) {
    // ---- best split of every open node of the level, one launch, one wait
    std::vector<int> open;  // indices into frontier, in histogram slot order
    for (size_t i = 0; i < frontier.size(); ++i)
      if (frontier[i].slot >= 0) open.push_back((int)i);
    std::sort(open.begin(), open.end(), [&](int a, int b) { return frontier[a].slot < frontier[b].slot; });
    const int n_open = (int)open.size();
    if (n_open == 0) break;
    for (int h0 = 0; h0 < n_open; h0 += kSplitMaxHists) {
      const int nh = n_open - h0 < kSplitMaxHists ? n_open - h0 : kSplitMaxHists;
      rc = found.enqueued(launch_split(hist_buf[cur] + (size_t)h0 * hist_elems, (int64_t)hist_elems, nh, lambda, min_child_hess,
                                       recs + h0, n_features, n_bins, s, found.device() + h0,
                                       level_sib.n > 0 ? &level_sib : nullptr));
      if (rc != GBDT_OK) return rc;
    }
    HIP_TRY(found.wait(s));
    if (!root_done) {
      const gbdt_split_t r = found[0];
      float sg = r.left_grad + r.right_grad, sh = r.left_hess + r.right_hess;
      if (r.feature < 0 && n_rows > 0) {  // no record carries the totals: sum feature 0's bins here
        std::vector<gbdt_bin_t> row((size_t)n_bins);
        HIP_TRY(hipMemcpyAsync(row.data(), hist_buf[cur], (size_t)n_bins * sizeof(gbdt_bin_t),
                               hipMemcpyDeviceToHost, s));
        HIP_TRY(hipStreamSynchronize(s));
        double g = 0.0, h = 0.0;
        for (const gbdt_bin_t& b : row) {
          g += b.grad;
          h += b.hess;
        }
        sg = (float)g;
        sh = (float)h;
      }
      fill_node(0, -1, r, sg, sh, (uint32_t)n_rows, 0);
      root_done = true;
    }
    // the records of the level's nodes (slot order = order of `open`)
    std::vector<gbdt_split_t> rec_of(frontier.size());
    for (int j = 0; j < n_open; ++j) {
      const gbdt_split_t& r = found[frontier[open[j]].slot];
      if (!split_fits(r, nodes_out[frontier[open[j]].node].count)) return GBDT_EHIP;
      rec_of[open[j]] = r;
      gbdt_tree_node_t& nd = nodes_out[frontier[open[j]].node];
      nd.feature = r.feature;
      nd.bin = r.bin;
      nd.gain = r.gain;
    }
    if (depth == max_depth) break;
    // ---- which nodes split, and where the partition finds their records
    std::vector<Entry> next;
    std::vector<int64_t> offs;          // positions of the entries of this level
    std::vector<int> splitting;         // indices into frontier
    std::vector<uint32_t> split_idx;    // by entry: slot of its record, or that there is none
    for (size_t i = 0; i < frontier.size(); ++i) {
      const gbdt_tree_node_t& nd = nodes_out[frontier[i].node];
      offs.push_back(nd.row_begin);
      split_idx.push_back(kNoSplitRecord);
      if (frontier[i].slot >= 0 && rec_of[i].feature >= 0 && rec_of[i].gain > min_split_gain) {
        split_idx.back() = (uint32_t)frontier[i].slot;
        splitting.push_back((int)i);
      }
    }
    offs.push_back(n_rows);
    if (splitting.empty()) break;
    const int nxt = cur ^ 1;
    // (the last level's rows go where the caller wants them)
    int32_t* rows_next = depth + 1 == max_depth && row_order_out ? row_order_out : rows_buf[nxt];
    rc = partition_rows_batch_impl(bin_matrix, n_rows, n_features, n_bins, rows_now, offs.data(),
                                   (int32_t)frontier.size(), recs, split_idx.data(), rows_next, nullptr, s);
    if (rc != GBDT_OK) return rc;
    rows_now = rows_next;
    // ---- children: node ids in the order of their parents' ids (the level's numbering),
    // histogram slots: the smaller children first (built), then the larger (by subtraction)
    std::vector<int> by_node = splitting;
    std::sort(by_node.begin(), by_node.end(), [&](int a, int b) { return frontier[a].node < frontier[b].node; });
    const int k = (int)by_node.size();
    std::vector<int64_t> small_offs = {0};
    std::vector<int> parent_slot((size_t)k);
    std::vector<uint32_t> small_seg((size_t)k);  // where a smaller child's rows begin
    std::vector<std::pair<Entry, Entry>> kids(frontier.size());
    for (int j = 0; j < k; ++j) {
      const int i = by_node[j];
      const int parent = frontier[i].node;
      const gbdt_split_t& r = rec_of[i];
      const int64_t begin = nodes_out[parent].row_begin;
      const int left = n_nodes, right = n_nodes + 1;
      n_nodes += 2;
      nodes_out[parent].left = left;
      nodes_out[parent].right = right;
      gbdt_split_t none;
      memset(&none, 0, sizeof none);
      none.feature = none.bin = -1;
      fill_node(left, parent, none, r.left_grad, r.left_hess, r.left_count, begin);
      fill_node(right, parent, none, r.right_grad, r.right_hess, r.right_count, begin + r.left_count);
      const bool left_small = r.left_count <= r.right_count;
      small_seg[j] = (uint32_t)(left_small ? begin : begin + r.left_count);
      small_offs.push_back(small_offs.back() + (left_small ? r.left_count : r.right_count));
      parent_slot[j] = frontier[i].slot;
      kids[i] = left_small ? std::make_pair(Entry{left, j}, Entry{right, k + j})
                           : std::make_pair(Entry{left, k + j}, Entry{right, j});
    }
    for (size_t i = 0; i < frontier.size(); ++i) {
      if (nodes_out[frontier[i].node].left >= 0) {
        next.push_back(kids[i].first);
        next.push_back(kids[i].second);
      } else {
        next.push_back(Entry{frontier[i].node, -1});  // a leaf from now on
      }
    }
    // ---- the smaller children's histograms in one batched build, straight from their segments of the rows
    rc = hist_build_batch_impl(bin_matrix, n_rows, n_features, n_bins, rows_now, small_offs.data(), k, grad,
                               hess, hist_buf[nxt], s, small_seg.data());
    if (rc != GBDT_OK) return rc;
    level_sib.pool = hist_buf[cur];
    level_sib.first = k;
    level_sib.n = k <= kSplitSiblings && 2 * k <= kSplitMaxHists ? k : 0;
    level_sib.keep = depth + 1 < max_depth;  // (nobody reads the last level's)
    for (int j = 0; j < level_sib.n; ++j) level_sib.parent_slot[j] = parent_slot[j];
    for (int j0 = 0; j0 < k && level_sib.n == 0; j0 += kSiblingTable) {
      SiblingTable t;
      const int ns = k - j0 < kSiblingTable ? k - j0 : kSiblingTable;
      for (int j = 0; j < ns; ++j) t.parent_slot[j] = parent_slot[j0 + j];
      hipLaunchKernelGGL(hist_siblings_kernel, dim3((unsigned)((hist_elems + 255) / 256), ns), dim3(256), 0, s,
                         (const gbdt_bin_t*)hist_buf[cur], (const gbdt_bin_t*)(hist_buf[nxt] + (size_t)j0 * hist_elems),
                         hist_buf[nxt] + (size_t)(k + j0) * hist_elems, (int32_t)hist_elems, t);
      HIP_TRY(hipGetLastError());
    }
    frontier.swap(next);
    cur = nxt;
  }
  *n_nodes_out = n_nodes;
  if (row_order_out && n_rows > 0 && !rows_now) {  // never split: the rows in their own order
    hipLaunchKernelGGL(row_iota_kernel, dim3((unsigned)((n_rows + 255) / 256)), dim3(256), 0, s, row_order_out, n_rows);
    HIP_TRY(hipGetLastError());
  } else if (row_order_out && n_rows > 0 && rows_now != row_order_out) {
    HIP_TRY(hipMemcpyAsync(row_order_out, rows_now, (size_t)n_rows * sizeof(int32_t), hipMemcpyDeviceToDevice, s));
  }
  return GBDT_OK;
}

int gbdt_debug_geometry(int32_t n_features, int32_t n_bins, int64_t n_leaf_rows, int32_t n_cus,
                        int64_t* out, int32_t n_out) {
  if (!out || n_out < 16 || n_features <= 0 || n_bins < 2 || n_bins > 256 || n_leaf_rows < 0)
    return GBDT_EINVAL;
  const BuildGeom g = make_geom(n_features, n_bins, n_leaf_rows, n_cus > 0 ? n_cus : 256, 0);
  const TilePlan& p = g.plan;
  const int64_t v[16] = {p.cap,         p.nib,          p.wm,          p.n_main,
                         p.wr,          p.row_bytes,    p.feat_bytes,  g.nt,
                         (int64_t)g.lds_bytes, g.wgs, g.unit_epochs, (int64_t)g.partial_words,
                         0,             0, 0, 0};
  for (int i = 0; i < 16; ++i) out[i] = v[i];
  return GBDT_OK;
}

int gbdt_debug_leaf_plan(int64_t n_rows, int32_t n_features, int32_t n_bins, int64_t n_leaf_rows, int32_t indexed,
                         int64_t* out, int32_t n_out) {
  if (!valid_shape(n_rows, n_features, n_bins) || n_leaf_rows < 0 || !out || n_out < 6) return GBDT_EINVAL;
  const bool wide = g_wide.load() != 0;
  const TilePlan p = make_tile_plan(n_features, n_bins);
  const bool halves = plan_halves(p, wide, rows_of_leaf(indexed != 0, n_leaf_rows, n_rows));
  const BuildGeom g = make_geom(n_features, n_bins, n_leaf_rows, device_cu_count(),
                                build_wg_per_cu(p.cap, indexed != 0, wide, halves), wide, halves);
  const UnitPlan u = plan_units(g, n_leaf_rows, indexed != 0, plan_line_tiles(n_rows), g_deterministic.load(), device_cu_count());
  const int64_t v[7] = {g.wgs, u.unit_epochs, u.first_epochs, u.fixed_stride, u.deal, g.one_unit_each, leaf_is_short(g, wide)};
  for (int i = 0; i < 7 && i < n_out; ++i) out[i] = v[i];
  return GBDT_OK;
}

int gbdt_debug_batch_plan(int32_t n_features, int32_t n_bins, const int64_t* leaf_offsets,
                          int32_t n_leaves, int32_t n_cus, int32_t wg_per_cu, int32_t* leaf_wgs_out,
                          int32_t* leaf_unit_epochs_out, int32_t* block_out, int32_t max_blocks) {
  if (n_features <= 0 || n_bins < 2 || n_bins > 256 || !leaf_offsets || n_leaves < 1 ||
      n_leaves > kBatchLeaves || n_cus <= 0 || wg_per_cu <= 0 || !leaf_wgs_out ||
      !leaf_unit_epochs_out || (!block_out && max_blocks > 0))
    return GBDT_EINVAL;
  for (int32_t l = 0; l < n_leaves; ++l)
    if (leaf_offsets[l + 1] < leaf_offsets[l]) return GBDT_EINVAL;
  const TilePlan p = make_tile_plan(n_features, n_bins);
  const int n_tiles = plan_n_tiles(p);
  const BatchPlan b = plan_batch(leaf_offsets, 0, n_leaves, n_cus, wg_per_cu, n_tiles);
  for (int32_t l = 0; l < n_leaves; ++l) {
    leaf_wgs_out[batch_leaf_no(b.leaf[l])] = (int32_t)batch_wgs(b.leaf[l]);
    leaf_unit_epochs_out[batch_leaf_no(b.leaf[l])] = (int32_t)batch_unit_epochs(b.leaf[l]);
  }
  const int64_t blocks = (int64_t)b.total_wgs * n_tiles;
  const int32_t deal =
      deal_order(plan_line_tiles(kPlanLinesMinRows), b.most_unit_epochs, blocks, n_cus, g_wide.load() != 0);
  for (int64_t i = 0; i < blocks && i < max_blocks; ++i) {
    const BatchBlock k = batch_block(b.leaf, n_leaves, p.wm, p.n_main, p.wr,
                                     deal, b.total_wgs, (uint32_t)i);
    block_out[3 * i] = (int32_t)batch_leaf_no(b.leaf[k.leaf]);
    block_out[3 * i + 1] = k.tile;
    block_out[3 * i + 2] = k.wg;
  }
  return (int)blocks;
}

int gbdt_debug_batch_is_short(int32_t n_features, int32_t n_bins, const int64_t* leaf_offsets, int32_t n_leaves, int32_t n_cus,
                              int32_t wg_per_cu) {
  if (n_features <= 0 || n_bins < 2 || n_bins > 256 || !leaf_offsets || n_leaves < 1 || n_leaves > kBatchLeaves || n_cus <= 0 ||
      wg_per_cu <= 0)
    return GBDT_EINVAL;
  for (int32_t l = 0; l < n_leaves; ++l)
    if (leaf_offsets[l + 1] < leaf_offsets[l]) return GBDT_EINVAL;
  const TilePlan p = make_tile_plan(n_features, n_bins);
  return batch_is_short(plan_batch(leaf_offsets, 0, n_leaves, n_cus, wg_per_cu, plan_n_tiles(p)), p.cap, g_wide.load() != 0) ? 1 : 0;
}

int gbdt_debug_block_map(int32_t n_features, int32_t n_bins, int64_t n_rows, int32_t cols, int32_t by_column,
                         int64_t* tile_out, int32_t* block_out, int32_t max_blocks) {
  if (n_rows < 0 || n_features <= 0 || n_bins < 2 || n_bins > 256 || cols < 1 || !tile_out || (!block_out && max_blocks > 0))
    return GBDT_EINVAL;
  const TilePlan p = make_tile_plan(n_features, n_bins);
  const int n_tiles = plan_n_tiles(p);
  const int32_t line_tiles = plan_line_tiles(n_rows);
  for (int32_t t = 0; t < n_tiles; ++t) {
    const TileAt at = plan_tile_at(p.wm, p.n_main, p.wr, n_rows, line_tiles, t);
    tile_out[2 * t] = at.off;
    tile_out[2 * t + 1] = at.stride;
  }
  const int64_t blocks = (int64_t)n_tiles * cols;
  if (blocks >= ((int64_t)1 << 31)) return GBDT_EUNSUPPORTED;
  const int32_t deal = deal_order(line_tiles, kUnitEpochs, blocks, 1, g_wide.load() != 0);
  for (int64_t i = 0; i < blocks && i < max_blocks; ++i) {
    const LineBlock b = line_block(p.wm, p.n_main, p.wr, deal, (uint32_t)cols, by_column != 0, (uint32_t)i);
    block_out[2 * i] = b.tile;
    block_out[2 * i + 1] = (int32_t)b.col;
  }
  return (int)blocks;
}

int gbdt_debug_half_blocks(int32_t n_features, int64_t n_rows, int32_t cols, int32_t by_column, int32_t* block_out,
                           int32_t max_blocks) {
  if (n_rows < 0 || n_features <= 0 || cols < 1 || (!block_out && max_blocks > 0)) return GBDT_EINVAL;
  const TilePlan p = make_tile_plan(n_features, 256);
  const int64_t blocks = (int64_t)plan_n_parts(p, true) * cols;
  if (blocks >= ((int64_t)1 << 31)) return GBDT_EUNSUPPORTED;
  const int32_t deal = deal_order(plan_line_tiles(n_rows), kUnitEpochs, blocks, 1, true);
  for (int64_t i = 0; i < blocks && i < max_blocks; ++i) {
    const HalfBlock b = half_block(p.wm, p.n_main, deal, (uint32_t)cols, by_column != 0, (uint32_t)i);
    block_out[3 * i] = b.tile;
    block_out[3 * i + 1] = b.half;
    block_out[3 * i + 2] = (int32_t)b.col;
  }
  return (int)blocks;
}

int gbdt_debug_gather_plan(const int64_t* leaf_offsets, int32_t n_leaves, int32_t* launch_out, int64_t* position_out) {
  if (!leaf_offsets || n_leaves < 1 || !launch_out || !position_out) return GBDT_EINVAL;
  for (int32_t l = 0; l < n_leaves; ++l)
    if (leaf_offsets[l + 1] < leaf_offsets[l] || leaf_offsets[l + 1] - leaf_offsets[l] >= ((int64_t)1 << 31)) return GBDT_EINVAL;
  int32_t launches = 0;
  GatherTable t;
  for (int32_t l0 = 0; l0 < n_leaves; l0 += t.n_lists, ++launches) {
    (void)fill_gather_table(leaf_offsets, nullptr, l0, n_leaves, &t);
    for (int32_t i = 0; i < t.n_lists; ++i) {
      launch_out[l0 + i] = launches;
      position_out[l0 + i] = leaf_offsets[l0] + (int64_t)t.first[i];
    }
  }
  return launches;
}

int gbdt_debug_host_blocks(int64_t* out) {
  if (!out) return GBDT_EINVAL;
  std::lock_guard<std::mutex> lk(g_rec_blocks.mu);
  out[0] = (int64_t)g_rec_blocks.idle.size();
  out[1] = (int64_t)g_rec_blocks.lost.size();
  out[2] = 0;
  for (const RecordBlock& b : g_rec_blocks.idle) out[2] = std::max(out[2], (int64_t)(b.n * sizeof(gbdt_split_t)));
  return GBDT_OK;
}

int gbdt_debug_fusion_plan(const uint32_t* levels, int32_t n_features, int32_t* col_out, int32_t* stride_out,
                           int32_t* n_cols_out) {
  if (!levels || n_features <= 0 || !col_out || !stride_out || !n_cols_out) return GBDT_EINVAL;
  std::vector<uint32_t> lv(levels, levels + n_features);
  for (uint32_t l : lv)
    if (l < 1 || l > (uint32_t)kFusedCap) return GBDT_EINVAL;
  std::vector<FusedCol> cols;
  std::vector<FusedFeat> feats;
  plan_fusion(lv, &cols, &feats);
  for (int32_t f = 0; f < n_features; ++f) {
    col_out[f] = feats[f].col;
    stride_out[f] = feats[f].stride;
  }
  *n_cols_out = (int32_t)cols.size();
  return GBDT_OK;
}

int64_t gbdt_debug_fuse_sample_rows(int64_t n_rows, int32_t n_features) {
  return n_rows > 0 && n_features > 0 ? fuse_sample_rows(n_rows, n_features) : 0;
}

int gbdt_debug_occupancy(int32_t n_bins, int32_t indexed) {
  if (n_bins < 2 || n_bins > 256) return GBDT_EINVAL;
  return build_wg_per_cu(n_bins <= 16 ? 16 : (n_bins <= 64 ? 64 : 256), indexed != 0);
}

int gbdt_debug_split_plan(int32_t n_features, int32_t n_bins, int32_t n_hists, int64_t* out, int32_t n_out) {
  if (!out || n_out < 4 || n_features <= 0 || n_bins < 2 || n_bins > 256 || n_hists < 1) return GBDT_EINVAL;
  const SplitGrouping g = split_grouping(n_features, n_bins, n_hists);
  out[0] = g.group;
  out[1] = g.passes;
  out[2] = g.n_wg;
  out[3] = g.waves;
  return GBDT_OK;
}

int gbdt_debug_partition_plan(int64_t n_leaf_rows, int64_t* out, int32_t n_out) {
  if (!out || n_out < 3 || n_leaf_rows < 1 || n_leaf_rows >= ((int64_t)1 << 32)) return GBDT_EINVAL;
  const PartGeom g = make_part_geom(n_leaf_rows);
  out[0] = g.rows_per_thread;
  out[1] = g.n_chunks;
  out[2] = (int64_t)g.bytes;
  return GBDT_OK;
}

int gbdt_debug_wide_pair(const float* first, const float* second, int32_t n, int64_t* out) {
  if (n < 1 || n > kEpochRows || !out || !first || !second) return GBDT_EINVAL;
  auto exponent = [n](const float* v) {  // (as scales_from has it)
    float sum = 0.0f;
    for (int32_t i = 0; i < n; ++i) sum += fabsf(v[i]);
    sum *= 1.001953125f;
    return epoch_scale_exp(__builtin_bit_cast(uint32_t, sum));
  };
  const int k = exponent(first), k2 = exponent(second), exp = wide_cell_exp(k, true);
  const bool pair = wide_pair(k, k2);
  uint64_t cell = 0, cell2 = 0;
  for (int32_t i = 0; i < n; ++i) {
    cell += ((uint64_t)wide_quantise(first[i], exp, 0) << kCountBits) + 1u;
    if (pair) cell2 += (uint64_t)wide_quantise(second[i], exp, k2 < k) << kCountBits;
  }
  out[0] = pair ? k2 - k : 2;
  out[1] = exp;
  out[2] = (int64_t)(cell + cell2) >> kCountBits;
  out[3] = (int64_t)cell2 >> kCountBits;
  out[4] = (int64_t)((cell + cell2) & ((1u << kCountBits) - 1u));
  return GBDT_OK;
}

int gbdt_debug_cell_sums(const int32_t* grad_q, const int32_t* hess_q, int32_t n, int64_t* out) {
  if (n < 0 || n > kEpochRows || !out || (n > 0 && (!grad_q || !hess_q))) return GBDT_EINVAL;
  uint64_t cell = 0;
  for (int32_t i = 0; i < n; ++i) {
    const CellWords w = cell_addend(grad_q[i], hess_q[i]);
    cell += ((uint64_t)w.hi << 32) | w.lo;
  }
  const CellSums s = cell_sums((uint32_t)cell, (uint32_t)(cell >> 32));
  out[0] = (int64_t)s.grad >> kSumPad;
  out[1] = (int64_t)s.hess >> kSumPad;
  out[2] = s.count;
  return GBDT_OK;
}

int gbdt_debug_locate(int32_t n_features, int32_t n_bins, int32_t feature, int32_t* tile_out,
                      int32_t* slot_out) {
  if (!tile_out || !slot_out || n_features <= 0 || n_bins < 2 || n_bins > 256 || feature < 0 ||
      feature >= n_features)
    return GBDT_EINVAL;
  const TilePlan p = make_tile_plan(n_features, n_bins);
  const FeatureSlot fs = plan_locate(p, feature);
  *tile_out = fs.tile;
  *slot_out = fs.slot;
  return GBDT_OK;
}

int gbdt_set_deterministic(int enable) {
  g_deterministic.store(enable != 0);
  return GBDT_OK;
}

int gbdt_set_wide_accumulation(int enable) {
  g_wide.store(enable != 0);
  return GBDT_OK;
}

int gbdt_calibration_copy(const void* src, void* dst, size_t bytes, void* stream) {
  if (!src || !dst || bytes == 0 || (bytes & 15u) != 0) return GBDT_EINVAL;
  if ((((uintptr_t)src) | ((uintptr_t)dst)) & 15u) return GBDT_EINVAL;
  hipLaunchKernelGGL(calibration_copy_kernel, dim3(device_cu_count() * 8), dim3(256), 0,
                     (hipStream_t)stream, (const uint4*)src, (uint4*)dst, bytes / 16);
  HIP_TRY(hipGetLastError());
  return GBDT_OK;
}

int gbdt_profile_enable(int enable) {
  std::lock_guard<std::mutex> lk(g_prof.mu);
  g_prof.on = enable != 0;
  return GBDT_OK;
}

int gbdt_profile_collect(double* build_kernel_ms_total, int64_t* n_launches) {
  if (!build_kernel_ms_total || !n_launches) return GBDT_EINVAL;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> pairs;
  {
    std::lock_guard<std::mutex> lk(g_prof.mu);
    pairs.swap(g_prof.pairs);
  }
  double total = 0.0;
  int rc = GBDT_OK;
  for (auto& pr : pairs) {
    float ms = 0.0f;
    hipError_t e = hipEventSynchronize(pr.second);
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, pr.first, pr.second);
    if (e != hipSuccess && rc == GBDT_OK) rc = hip_fail(e, "hipEventElapsedTime");
    total += ms;
    (void)hipEventDestroy(pr.first);
    (void)hipEventDestroy(pr.second);
  }
  *build_kernel_ms_total = total;
  *n_launches = (int64_t)pairs.size();
  return rc;
}

int gbdt_profile_durations(double* ms_out, int64_t capacity, int64_t* n_launches) {
  if (!n_launches || capacity < 0 || (capacity > 0 && !ms_out)) return GBDT_EINVAL;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> pairs;
  {
    std::lock_guard<std::mutex> lk(g_prof.mu);
    pairs.swap(g_prof.pairs);
  }
  int rc = GBDT_OK;
  int64_t i = 0;
  for (auto& pr : pairs) {
    float ms = 0.0f;
    hipError_t e = hipEventSynchronize(pr.second);
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, pr.first, pr.second);
    if (e != hipSuccess && rc == GBDT_OK) rc = hip_fail(e, "hipEventElapsedTime");
    if (i < capacity) ms_out[i] = ms;
    ++i;
    (void)hipEventDestroy(pr.first);
    (void)hipEventDestroy(pr.second);
  }
  *n_launches = i;
  return rc;
}

int gbdt_reset(void) {
  // everything enqueued so far must be done before buffers go away and counters are cleared
  HIP_TRY(hipDeviceSynchronize());
  {
    std::lock_guard<std::mutex> lk(g_ws.mu);
    for (void* q : g_ws.retired) (void)hipFree(q);
    g_ws.retired.clear();
    if (g_ws.own) (void)hipFree(g_ws.own);
    g_ws.own = nullptr;
    g_ws.own_bytes = 0;
    g_ws.own_device = -1;
    g_ws.zeroed = nullptr;  // a caller's buffer stays registered; its counters are zeroed by the next build
  }
  {
    std::lock_guard<std::mutex> lk(g_prof.mu);
    for (auto& pr : g_prof.pairs) {
      (void)hipEventDestroy(pr.first);
      (void)hipEventDestroy(pr.second);
    }
    g_prof.pairs.clear();
  }
  {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_rec_blocks.mu);
    for (auto* list : {&g_rec_blocks.idle, &g_rec_blocks.lost}) {  // (of this device: no other has been waited for)
      auto done = std::partition(list->begin(), list->end(), [&](const RecordBlock& b) { return b.device != dev; });
      for (auto it = done; it != list->end(); ++it) (void)hipHostFree(it->host);
      list->erase(done, list->end());
    }
  }
  (void)hipGetLastError();
  // the split search's tickets: a launch that failed half-way may have left some counted
  hipLaunchKernelGGL(split_tickets_zero_kernel, dim3(kSplitMaxHists / 256), dim3(256), 0, nullptr);
  HIP_TRY(hipGetLastError());
  HIP_TRY(hipDeviceSynchronize());
  g_hip_err[0] = 0;
  return GBDT_OK;
}

const char* gbdt_strerror(int code) {
  switch (code) {
    case GBDT_OK: return "ok";
    case GBDT_EINVAL: return "invalid argument";
    case GBDT_EUNSUPPORTED: return "unsupported problem size";
    case GBDT_EHIP: return "HIP runtime error";
    case GBDT_ENOMEM: return "workspace allocation failed or too small";
    default: return "unknown error code";
  }
}

const char* gbdt_last_hip_error(void) { return g_hip_err; }

}  // extern "C"
