// Best-split search over bin boundaries (Sec. 3.3).  Included by gbdt_hist.hip only.
#ifndef GBDT_SPLIT_KERNELS_H_
#define GBDT_SPLIT_KERNELS_H_

#include <hip/hip_runtime.h>

#include <stdint.h>
#include <string.h>

#include <type_traits>

#include "../../include/gbdt_hist.h"

namespace {

// ------------------------------------------------------------------ split kernels

struct SplitCand {
  double gain;
  double gl, hl, gr, hr;
  uint32_t nl, nr;
  int32_t feature;  // -1: no admissible threshold among this workgroup's features
  int32_t bin;
};

static_assert(sizeof(SplitCand) == 7 * 8, "a candidate is moved as 7 64-bit words");

constexpr int kSplitMaxWaves = 16;  // wavefronts of a workgroup at most
constexpr int kSplitMaxHists = 32768;  // histograms per launch (grid.y)

// One ticket counter per histogram of a launch: the workgroups of a histogram count
// themselves off, and the last of them sets the counter back to zero, so the counters
// need no resetting between launches (zero when the module is loaded).
__device__ unsigned int g_split_ticket[kSplitMaxHists];
// The counters of neighbouring histograms lie kSplitTicketStride words apart: every workgroup of a
// launch adds to one of them with a device-scope atomic, those are carried out one after the
// other where the word's memory channel is, and with the counters of a launch side by side the
// whole launch queued at one channel (measured: 14 ns per workgroup, 28 us for 8 x 250 of them).
constexpr int kSplitTicketStride = 64;
__device__ __forceinline__ unsigned int* split_ticket(unsigned int y) {
  constexpr unsigned int lines = kSplitMaxHists / kSplitTicketStride;
  return &g_split_ticket[(y % lines) * kSplitTicketStride + y / lines];
}

// Sets every ticket counter back to zero (gbdt_reset: after a launch that did not complete).
__global__ void __launch_bounds__(256) split_tickets_zero_kernel() {
  g_split_ticket[blockIdx.x * 256 + threadIdx.x] = 0u;
}

// Candidates cross from the workgroups that write them to the one that reduces them,
// possibly on another XCD with its own L2: they are moved with device-scope atomic
// accesses (which bypass the caches that are not coherent across XCDs), inside the
// release / acquire fences around the ticket.
__device__ __forceinline__ void store_cand(SplitCand* dst, const SplitCand& c) {
  unsigned long long w[7];
  memcpy(w, &c, sizeof c);
  unsigned long long* d = reinterpret_cast<unsigned long long*>(dst);
#pragma unroll
  for (int i = 0; i < 7; ++i) __hip_atomic_store(d + i, w[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long load_cand_word(const SplitCand* src, int i) {
  unsigned long long* p = const_cast<unsigned long long*>(reinterpret_cast<const unsigned long long*>(src));
  return __hip_atomic_load(p + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// What the arg-max looks at: the gain (word 0) and the feature (word 6, with the bin).
__device__ __forceinline__ void load_cand_key(const SplitCand* src, double* gain, int32_t* feature) {
  const unsigned long long w0 = load_cand_word(src, 0), w6 = load_cand_word(src, 6);
  memcpy(gain, &w0, sizeof *gain);
  *feature = (int32_t)(uint32_t)(w6 & 0xffffffffull);
}
__device__ __forceinline__ SplitCand load_cand(const SplitCand* src) {
  unsigned long long w[7];
#pragma unroll
  for (int i = 0; i < 7; ++i) w[i] = load_cand_word(src, i);
  SplitCand c;
  memcpy(&c, w, sizeof c);
  return c;
}
// How a wavefront holds histogram rows: a lane has kSplitBins consecutive bins of a feature, so a row takes
// 1 << lane_bits lanes (4, 8, .. 64) and a wavefront 64 >> lane_bits rows at a time, a STEP.
constexpr int kSplitBins = 4;
__host__ __device__ inline int split_lane_bits(int n_bins) {
  int b = 2;
  while ((kSplitBins << b) < n_bins) ++b;
  return b;
}

// Data of another lane of the wavefront, by DPP; lanes without a source, and rows of 16 lanes that ROW_MASK
// leaves out, get 0.
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ double dpp_or_zero(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROW_MASK, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)((unsigned long long)b >> 32), CTRL, ROW_MASK, 0xf, true);
  return __longlong_as_double((long long)(((unsigned long long)(uint32_t)hi << 32) | (uint32_t)lo));
}
__device__ __forceinline__ double and_mask(double v, uint32_t m) {  // v, or 0 where m is 0 (else m is all ones)
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  return __longlong_as_double(
      (long long)(((unsigned long long)((uint32_t)(b >> 32) & m) << 32) | ((uint32_t)b & m)));
}

// The lanes of a row: shifts and sums over them.  (Rows of 16 lanes and more are what DPP shifts keep apart by
// themselves; shorter ones mask what comes from the row before.)
template <int LB>
struct RowLanes {
  uint32_t from1, from2, from4;  // all ones where the lane 1, 2, 4 places before is of the same row
  __device__ __forceinline__ explicit RowLanes(int lane) {
    const int l = lane & ((1 << LB) - 1);
    from1 = l >= 1 ? ~0u : 0u;
    from2 = l >= 2 ? ~0u : 0u;
    from4 = l >= 4 ? ~0u : 0u;
  }
  // sum over the row's lanes up to and with this one
  __device__ __forceinline__ double prefix(double t) const {
    if constexpr (LB >= 4) {
      t += dpp_or_zero<0x111>(t);  // row_shr:1, 2, 4, 8
      t += dpp_or_zero<0x112>(t);
      t += dpp_or_zero<0x114>(t);
      t += dpp_or_zero<0x118>(t);
      if constexpr (LB >= 5) t += dpp_or_zero<0x142, 0xa>(t);  // row_bcast15
      if constexpr (LB >= 6) t += dpp_or_zero<0x143, 0xc>(t);  // row_bcast31
    } else {
      t += and_mask(dpp_or_zero<0x111>(t), from1);
      t += and_mask(dpp_or_zero<0x112>(t), from2);
      if constexpr (LB >= 3) t += and_mask(dpp_or_zero<0x114>(t), from4);
    }
    return t;
  }
  // the value of the lane before, 0 in a row's first lane
  __device__ __forceinline__ double before(double t) const {
    if constexpr (LB == 4) return dpp_or_zero<0x111>(t);  // row_shr:1
    if constexpr (LB == 6) return dpp_or_zero<0x138>(t);  // wave_shr:1
    return and_mask(dpp_or_zero<0x138>(t), from1);
  }
  // the value of the row's last lane
  __device__ __forceinline__ double last(double t, int lane) const {
    const long long b = __double_as_longlong(t);
    const int lo = (int)(uint32_t)b, hi = (int)(uint32_t)((unsigned long long)b >> 32);
    int rl, rh;
    if constexpr (LB == 6) {
      rl = __builtin_amdgcn_readlane(lo, 63);
      rh = __builtin_amdgcn_readlane(hi, 63);
    } else if constexpr (LB == 5) {
      const int l0 = __builtin_amdgcn_readlane(lo, 31), l1 = __builtin_amdgcn_readlane(lo, 63);
      const int h0 = __builtin_amdgcn_readlane(hi, 31), h1 = __builtin_amdgcn_readlane(hi, 63);
      rl = lane < 32 ? l0 : l1;
      rh = lane < 32 ? h0 : h1;
    } else if constexpr (LB == 4) {
      rl = __builtin_amdgcn_update_dpp(0, lo, 0x15f, 0xf, 0xf, false);  // row_newbcast:15
      rh = __builtin_amdgcn_update_dpp(0, hi, 0x15f, 0xf, 0xf, false);
    } else if constexpr (LB == 3) {  // lanes 0..7 of a row of 16 take lane 7, the others lane 15
      rl = __builtin_amdgcn_update_dpp(0, lo, 0x157, 0xf, 0x3, false);
      rl = __builtin_amdgcn_update_dpp(rl, lo, 0x15f, 0xf, 0xc, false);
      rh = __builtin_amdgcn_update_dpp(0, hi, 0x157, 0xf, 0x3, false);
      rh = __builtin_amdgcn_update_dpp(rh, hi, 0x15f, 0xf, 0xc, false);
    } else {
      rl = __builtin_amdgcn_update_dpp(0, lo, 0xff, 0xf, 0xf, false);  // quad_perm [3,3,3,3]
      rh = __builtin_amdgcn_update_dpp(0, hi, 0xff, 0xf, 0xf, false);
    }
    return __longlong_as_double((long long)(((unsigned long long)(uint32_t)rh << 32) | (uint32_t)rl));
  }
};

// Largest value / smallest index over the wavefront, in every lane.  (NaN is passed over.)
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_max(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = (int)(uint32_t)b, hi = (int)(uint32_t)((unsigned long long)b >> 32);
  const int l2 = __builtin_amdgcn_update_dpp(lo, lo, CTRL, ROW_MASK, 0xf, false);
  const int h2 = __builtin_amdgcn_update_dpp(hi, hi, CTRL, ROW_MASK, 0xf, false);
  return fmax(v, __longlong_as_double((long long)(((unsigned long long)(uint32_t)h2 << 32) | (uint32_t)l2)));
}
__device__ __forceinline__ double wave_max(double v) {
  v = dpp_max<0xb1, 0xf>(v);   // quad_perm [1,0,3,2]
  v = dpp_max<0x4e, 0xf>(v);   // quad_perm [2,3,0,1]
  v = dpp_max<0x141, 0xf>(v);  // row_half_mirror
  v = dpp_max<0x140, 0xf>(v);  // row_mirror
  v = dpp_max<0x142, 0xa>(v);  // row_bcast15
  v = dpp_max<0x143, 0xc>(v);  // row_bcast31
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(uint32_t)b, 63);
  const int hi = __builtin_amdgcn_readlane((int)(uint32_t)((unsigned long long)b >> 32), 63);
  return __longlong_as_double((long long)(((unsigned long long)(uint32_t)hi << 32) | (uint32_t)lo));
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_min(int v) {
  const int o = __builtin_amdgcn_update_dpp(v, v, CTRL, ROW_MASK, 0xf, false);
  return o < v ? o : v;
}
__device__ __forceinline__ int wave_min(int v) {
  v = dpp_min<0xb1, 0xf>(v);
  v = dpp_min<0x4e, 0xf>(v);
  v = dpp_min<0x141, 0xf>(v);
  v = dpp_min<0x140, 0xf>(v);
  v = dpp_min<0x142, 0xa>(v);
  v = dpp_min<0x143, 0xc>(v);
  return __builtin_amdgcn_readlane(v, 63);
}
// A gain that is no number (0 / 0: lambda = 0 and a side without gradient and hessian) loses against every number, in a lane,
// a wavefront, a workgroup and between them, so a search does not depend on how its steps are dealt out.
__device__ __forceinline__ bool gain_beats(double gain, double best) { return !(best >= gain) && gain == gain; }
// The index of the wavefront's best (gain, index) under the order "larger gain, then smaller index"
// (index < 0: no candidate); -1 if no lane has one.
__device__ __forceinline__ int32_t wave_argmax(double gain, int32_t idx) {
  const double top = wave_max(idx >= 0 ? gain : -INFINITY);
  bool mine = idx >= 0 && gain == top;
  if (__ballot(mine) == 0ull) mine = idx >= 0;
  const int32_t best = wave_min(mine ? idx : 0x7fffffff);
  return best == 0x7fffffff ? -1 : best;
}

// Gain scan of Sec. 3.3.  A wavefront takes a step of rows at a time, all in registers, no local memory and no barriers:
//  1. Lanes fetch their kSplitBins bins.
//  2. Running sums of gradient, hessian and count in fp64.  The result has to be that of the sum strictly from left
//     to right (it decides which thresholds tie exactly), so the sums are formed in parallel -- within a lane,
//     then over the row's lanes -- and CHECKED: if p[i] == p[i - 1] + v[i] holds in fp64 for every bin, then
//     p is that sum, by induction.  It holds whenever no addition rounds, i.e. unless the row's
//     values span more than some 20 binary orders of magnitude; then the lanes correct their sums until it does, 2 to
//     6 turns for most rows.  (Counts never round.)
//  3. The gains.  Divisions are the expensive part, and nearly all of them lose: an approximation by one reciprocal with
//     a bound of its error rules out what cannot beat the best gain the wavefront knows, and only
//     the rest is divided out.
// Feature totals are the prefix at the last bin, right = total - left, a threshold is
// admissible when both sides hold >= 1 sample and >= min_child_hess of hessian (so the last bin never is).
//  4. Arg-max over the wavefront, then over the workgroup's wavefronts, and where a histogram has several workgroups, over
//     those: the one that finishes last (a ticket taken after its own candidate is written; nobody waits) reduces
//     the candidates of all to the histogram's split record: workgroups hold ascending features,
//     so "smaller candidate index" is "smaller feature".
// Bound by vector work (about 240 instructions a step) and, with many histograms, by reading them: 64 histograms of 2,000 x 63
// take 23.6 us, 4.1 TB/s, 256 of them 75 (5.2 TB/s); a lone one 6.2.  Where the sums of every row round: 64 of 2,000 x 63 36 us, 64 of 500 x
// 255 54 instead of 25 (41 and 93 with one lane after the other summing from left to right, 16 and 64 turns), a lone 28 x 255 6.8
// instead of 5.2.  (A workgroup used to stage up to 16
// features in local memory, one wavefront ran their sums one bin after the other while the others waited, and
// every threshold was divided out: 50.6, 156 and 9.8 us, 79 for 500 x 255 and 8.9 for 28 x 255, whatever the sums.)  Lanes of four bins, not one, because the sums over lanes are most of the
// work: 2 vector instructions a bin and statistic for them so, 6 with 64 lanes a row.  The next step's rows
// are requested before the present ones are used: 25.8 us without.
// grid.y = histogram of the call; histogram y starts hist_stride bins after histogram
// y - 1 (the stride may be negative: any two histograms of a pool can be searched in
// one launch).  mirror (may be NULL): a second place for the records, page-locked host
// memory that the device can write, so that a caller who must look at them on the host
// needs no copy after the kernel, only to wait for it.
// sib (sib.n may be 0): histograms sib.first .. sib.first + sib.n - 1 of the call are siblings
// by subtraction that do not exist yet: histogram sib.first + j is first formed, element by
// element as hist_subtract_kernel does it, as (pool histogram parent_slot[j]) - (histogram j of
// the call, the built child), written to its place (unless nobody will read it: keep == 0) and searched in the
// same pass: every (feature, bin) is read by exactly one workgroup, which also writes the difference.
constexpr int kSplitSiblings = 512;
struct SplitSiblings {
  const gbdt_bin_t* pool;  // histograms of hist_elems bins each
  int32_t first, n;
  int32_t keep;
  int32_t parent_slot[kSplitSiblings];
};
struct NoSiblings {};  // (a launch without siblings does not carry the table)

template <int LB, bool SHORT, typename SIB>
__global__ void __launch_bounds__(64 * kSplitMaxWaves)
split_gain_kernel(gbdt_bin_t* hist, int64_t hist_stride, int32_t n_features,
                  int32_t n_bins, int32_t wg_steps, double lambda, double min_child_hess,
                  SplitCand* __restrict__ cand, gbdt_split_t* __restrict__ out,
                  gbdt_split_t* __restrict__ mirror, SIB sib) {
  constexpr int kRows = 64 >> LB;
  constexpr int K = kSplitBins;
  __shared__ SplitCand s_cand[kSplitMaxWaves];
  __shared__ int32_t s_pair[kSplitMaxWaves];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int n_waves = (int)blockDim.x >> 6;
  bool is_sib = false;
  const gbdt_bin_t *built = nullptr, *sib_parent = nullptr;  // the sibling's built twin, and their parent
  if constexpr (std::is_same_v<SIB, SplitSiblings>) {
    const int32_t sib_j = (int32_t)blockIdx.y - sib.first;
    is_sib = sib_j >= 0 && sib_j < sib.n;
    if (is_sib) {
      built = hist + (int64_t)sib_j * hist_stride;
      sib_parent = sib.pool + (int64_t)sib.parent_slot[sib_j] * hist_stride;
    }
  }
  hist += (int64_t)blockIdx.y * hist_stride;
  const int B = n_bins;
  const RowLanes<LB> row_lanes(lane);
  const int bin0 = K * (lane & ((1 << LB) - 1));  // this lane's first bin
  const int row = lane >> LB;
  // Of a row that ends inside its K bins a lane fetches the row's last K, so that no load leaves the row, and the
  // first `skip` of them, which the lane before has, count as zero.  Lanes past the row's end skip all.
  const int past = bin0 + K - B;
  const int skip = past < 0 ? 0 : (past < K ? past : K);
  const bool whole = B == (K << LB);  // (then no lane skips anything)
  const int first_bin = SHORT ? 0 : (bin0 - skip < B - K ? bin0 - skip : B - K);

  const int32_t n_steps = (n_features + kRows - 1) / kRows;
  const int32_t step0 = (int32_t)blockIdx.x * wg_steps;
  const int32_t f_first = step0 * kRows;
  const int32_t step_end = n_steps - step0 < wg_steps ? n_steps : step0 + wg_steps;

  auto row_of = [&](int32_t step) {  // (rows past the last feature: the last one again, counted as zeros)
    const int32_t f = step * kRows + row;
    return (size_t)(f < n_features ? f : n_features - 1) * B + first_bin;
  };
  auto fetch = [&](const gbdt_bin_t* from, size_t at, gbdt_bin_t (&v)[K]) {
    if constexpr (!SHORT) {
      __builtin_memcpy(v, from + at, sizeof v);
    } else {  // two or three bins: the one lane of a row that has any keeps them in its last places
#pragma unroll
      for (int k = 0; k < K; ++k) v[k] = from[at + (k < K - B ? 0 : k - (K - B))];
    }
  };

  // The approximation takes both quotients as one, good to about 2^-48 of their sum while the denominators are
  // positive -- as they are where a side's hessian has to be.
  constexpr double kSlack = 0x1p-40;
  const bool positive = min_child_hess > 0.0;
  auto arrives = [](double sum, double claim) { return (sum == claim) | ((sum != sum) & (claim != claim)); };
  double bound = -INFINITY;  // some threshold the wavefront has seen gains at least this
  // this lane's best pair with everything the record needs
  double best_gain = 0.0, best_gl = 0.0, best_hl = 0.0, best_nl = 0.0, best_g = 0.0, best_h = 0.0, best_n = 0.0;
  int32_t best_pair = -1;  // (feature - f_first) * (B - 1) + bin, ascending in (feature, bin)
  gbdt_bin_t next[K];  // the next step's
  fetch(is_sib ? built : hist, row_of(step0 + wave), next);
  for (int32_t step = step0 + wave; step < step_end; step += n_waves) {
    gbdt_bin_t v[K];
    const size_t at = row_of(step);
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = next[k];
    fetch(is_sib ? built : hist, row_of(step + n_waves), next);
    // places of this lane that hold no bin of their own
    const int none = (step + 1) * kRows <= n_features || step * kRows + row < n_features ? skip : K;
    if (is_sib) {
      gbdt_bin_t q[K];
      fetch(sib_parent, at, q);
#pragma unroll
      for (int k = 0; k < K; ++k) {
        v[k].grad = q[k].grad - v[k].grad;
        v[k].hess = q[k].hess - v[k].hess;
        v[k].count = q[k].count - v[k].count;
      }
      if constexpr (std::is_same_v<SIB, SplitSiblings>) {
        if (sib.keep && none < K) {  // (where lanes overlap they write the same)
          if constexpr (!SHORT) {
            __builtin_memcpy(hist + at, v, sizeof v);
          } else {
#pragma unroll
            for (int k = 0; k < K; ++k) hist[at + (k < K - B ? 0 : k - (K - B))] = v[k];
          }
        }
      }
    }
    if (!whole || (step + 1) * kRows > n_features) {
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (k < none) v[k] = gbdt_bin_t{0.0f, 0.0f, 0u};
    }
    // running sums
    double pg[K], ph[K], pn[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      pg[k] = (k ? pg[k - 1] : 0.0) + (double)v[k].grad;
      ph[k] = (k ? ph[k - 1] : 0.0) + (double)v[k].hess;
      pn[k] = (k ? pn[k - 1] : 0.0) + (double)v[k].count;
    }
    const double bg = row_lanes.before(row_lanes.prefix(pg[K - 1]));
    const double bh = row_lanes.before(row_lanes.prefix(ph[K - 1]));
    const double bn = row_lanes.before(row_lanes.prefix(pn[K - 1]));
#pragma unroll
    for (int k = 0; k < K; ++k) {
      pg[k] += bg;
      ph[k] += bh;
      pn[k] += bn;
    }
    bool same = row_lanes.before(pg[K - 1]) == bg;
    same &= row_lanes.before(ph[K - 1]) == bh;
#pragma unroll
    for (int k = 1; k < K; ++k) {
      same &= pg[k - 1] + (double)v[k].grad == pg[k];
      same &= ph[k - 1] + (double)v[k].hess == ph[k];
    }
    if (__ballot(!same) != 0ull) {
      // A lane's sums at its last bin are what it claims.  A turn sums every lane's bins onto the claim of the lane before; if
      // all arrive at their claims, those are the sums from left to right.  Else claims move by what they and the claims
      // before them were off.  (After turn i the row's lanes 0 .. i are right whatever the values are.)
#pragma unroll 1
      for (int turn = 0; turn < (1 << LB); ++turn) {
        double g = row_lanes.before(pg[K - 1]), h = row_lanes.before(ph[K - 1]);
#pragma unroll
        for (int k = 0; k < K - 1; ++k) {
          pg[k] = g += (double)v[k].grad;
          ph[k] = h += (double)v[k].hess;
        }
        g += (double)v[K - 1].grad;
        h += (double)v[K - 1].hess;
        const double off_g = arrives(g, pg[K - 1]) ? 0.0 : g - pg[K - 1], off_h = arrives(h, ph[K - 1]) ? 0.0 : h - ph[K - 1];
        if (__ballot(!(off_g == 0.0 && off_h == 0.0)) == 0ull) break;
        pg[K - 1] = g + row_lanes.before(row_lanes.prefix(off_g));
        ph[K - 1] = h + row_lanes.before(row_lanes.prefix(off_h));
      }
    }
    const double G = row_lanes.last(pg[K - 1], lane), H = row_lanes.last(ph[K - 1], lane);
    const double N = row_lanes.last(pn[K - 1], lane);

    // what a threshold gains at most
    const double hp = H + lambda;
    double rp = __builtin_amdgcn_rcp(hp);
    rp = fma(rp, fma(-hp, rp, 1.0), rp);
    const double parent_about = G * G * rp, parent_least = parent_about * (1.0 - kSlack);
    double most[K];
    bool ok[K], any = false;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const double GL = pg[k], HL = ph[k], GR = G - GL, HR = H - HL;
      ok[k] = pn[k] >= 1.0 && N - pn[k] >= 1.0 && HL >= min_child_hess && HR >= min_child_hess && k >= none;
      const double a = HL + lambda, b = HR + lambda, ab = a * b;
      double r = __builtin_amdgcn_rcp(ab);
      r = fma(r, fma(-ab, r, 1.0), r);
      most[k] = fma(fma(GL * GL, b, GR * GR * a) * r, 1.0 + kSlack, -parent_least);
      any = any || (ok[k] && (!positive || !(most[k] < bound)));
    }
    if (__ballot(any) != 0ull) {
      if (positive) {  // what some threshold gains for certain
        double top = -INFINITY;
#pragma unroll
        for (int k = 0; k < K; ++k) top = ok[k] ? fmax(top, most[k]) : top;
        bound = fmax(bound, wave_max(top - 8.0 * kSlack * (fabs(top) + parent_about)));
      }
      const double parent = __ddiv_rn(__dmul_rn(G, G), hp);
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const bool divide = ok[k] && (!positive || !(most[k] < bound));  // (true where most[k] is no number)
        if (__ballot(divide) == 0ull) continue;
        if (divide) {
          const double GL = pg[k], HL = ph[k], GR = G - GL, HR = H - HL;
          const double lt = __ddiv_rn(__dmul_rn(GL, GL), HL + lambda);
          const double rt = __ddiv_rn(__dmul_rn(GR, GR), HR + lambda);
          const double gain = __dsub_rn(__dadd_rn(lt, rt), parent);
          if (best_pair < 0 || gain_beats(gain, best_gain)) {  // pairs ascend: ties keep the earlier pair
            best_gain = gain;
            best_pair = (step * kRows + row - f_first) * (B - 1) + bin0 - skip + k;
            best_gl = GL;
            best_hl = HL;
            best_nl = pn[k];
            best_g = G;
            best_h = H;
            best_n = N;
          }
        }
      }
    }
  }

  // the wavefront's best pair, then the workgroup's
  {
    const int32_t top = wave_argmax(best_gain, best_pair);
    if (top < 0 ? lane == 0 : best_pair == top) {
      SplitCand c;
      if (top < 0) {
        c.gain = 0.0;
        c.gl = c.hl = c.gr = c.hr = 0.0;
        c.nl = c.nr = 0;
        c.feature = -1;
        c.bin = -1;
      } else {
        const int fl = top / (B - 1);
        c.gain = best_gain;
        c.gl = best_gl;
        c.hl = best_hl;
        c.nl = (uint32_t)best_nl;
        c.gr = best_g - best_gl;
        c.hr = best_h - best_hl;
        c.nr = (uint32_t)(best_n - best_nl);
        c.feature = f_first + fl;
        c.bin = top - fl * (B - 1);
      }
      s_cand[wave] = c;
      s_pair[wave] = top;
    }
  }
  __syncthreads();
  if (wave != 0) return;  // the first wavefront does the rest
  const int32_t my_pair = lane < n_waves ? s_pair[lane] : -1;
  const int32_t top = wave_argmax(lane < n_waves ? s_cand[lane & (kSplitMaxWaves - 1)].gain : 0.0, my_pair);
  const bool writer = top < 0 ? lane == 0 : my_pair == top;
  auto write_record = [&](const SplitCand& c) {
    gbdt_split_t r;
    r.feature = c.feature;
    r.bin = c.bin;
    r.gain = (float)c.gain;
    r.left_grad = (float)c.gl;
    r.left_hess = (float)c.hl;
    r.left_count = c.nl;
    r.right_grad = (float)c.gr;
    r.right_hess = (float)c.hr;
    r.right_count = c.nr;
    out[blockIdx.y] = r;
    if (mirror) mirror[blockIdx.y] = r;
  };
  const int32_t n_cand = (int32_t)gridDim.x;
  if (n_cand == 1) {  // the histogram's only workgroup
    if (writer) write_record(s_cand[lane]);
    return;
  }
  cand += (size_t)blockIdx.y * gridDim.x;
  bool last = false;
  if (writer) {
    store_cand(cand + blockIdx.x, s_cand[lane]);
    // HARDWARE ASSUMPTION (gfx942 / gfx950, not the language's memory model): a device-scope
    // atomic store is written through to the point where the other XCDs' device-scope atomic
    // loads read it, and is acknowledged (vmcnt) only then.  Waiting for the candidate's
    // stores (vmcnt(0)) before taking the ticket is therefore all the release this hand-off
    // needs, and the reader needs no acquire because it reads the candidates with device-scope
    // atomic loads only.  A release / acquire pair in the language's sense would also write back
    // and invalidate every line of the L2, which costs tens of microseconds here -- several
    // times the whole kernel.  tests/test_gpu_robustness.py runs 20 launches of 64 histograms of 16 workgroups
    // that hand off so, and launches of up to 256 a histogram; every split test of more than one workgroup goes through it.  On a
    // part where the assumption did not hold those tests would show stale candidates.
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0); expcnt, lgkmcnt untouched
    unsigned int* ticket = split_ticket(blockIdx.y);
    const unsigned int old = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last = old == gridDim.x - 1;
    if (last)  // back to zero for the next launch
      __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (__ballot(last) == 0ull) return;
  // The ticket's value has arrived, so every other workgroup's candidate was acknowledged
  // before its ticket; the loads below are device-scope atomics and bypass stale caches.

  // ---- the histogram's last workgroup: arg-max over all candidates.  (Two round trips to the other workgroups'
  // results: the keys of all candidates, then the winner's record, which its owner fetches and writes.
  // Fetching whole candidates at once saves the second, but 56 bytes apart seven words of each take longer than that.)
  double bg = 0.0;
  int32_t bi = -1;
  for (int32_t i = lane; i < n_cand; i += 64) {
    double gain;
    int32_t feature;
    load_cand_key(cand + i, &gain, &feature);
    if (feature >= 0 && (bi < 0 || gain_beats(gain, bg))) {  // i ascends, so ties keep the smaller feature
      bg = gain;
      bi = i;
    }
  }
  const int32_t won = wave_argmax(bg, bi);
  if (won < 0 ? lane == 0 : bi == won) {
    if (won < 0) {
      write_record(s_cand[0]);  // (no workgroup has an admissible threshold, this one included)
    } else {
      write_record(load_cand(cand + won));
    }
  }
}

}  // namespace

#endif  // GBDT_SPLIT_KERNELS_H_
