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

constexpr int kSplitThreads = 256;
constexpr int kSplitLdsBudget = 48 * 1024;
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
// LDS bytes one feature needs in split_gain_kernel: fp64 running sums of gradient,
// hessian and count per bin (bins padded to a multiple of kSplitBlock), + the feature's parent term.
// A row is two doubles longer than that: the prefix pass walks down all rows of a group at once,
// 16 bytes per lane, and with rows an odd multiple of 16 bytes apart the lanes fall on different banks
// (with rows a multiple of 128 bytes apart, as they were, all of them fell on the same: 16 features
// x 64 bins took 6,100 cycles there).
constexpr int kSplitBlock = 16;  // bins the prefix loop adds per register block
__host__ __device__ inline int split_padded_bins(int n_bins) { return (n_bins + kSplitBlock - 1) & ~(kSplitBlock - 1); }
__host__ __device__ inline int split_row(int n_bins) { return split_padded_bins(n_bins) + 2; }
__host__ __device__ inline int split_feature_bytes(int n_bins) { return 24 * split_row(n_bins) + 8; }

// How the workgroup's wavefronts walk over the (feature, bin) pairs of a group, in steps of 64: up to 64 bins
// a step is 64 / lanes rows side by side (lanes = the bins rounded up to a power of two), beyond that a
// row takes `chunks` steps.  No division per thread, and a step's loads are whole rows.
constexpr int kSplitSteps = 8;  // steps a wavefront takes of a group at most: 32 steps a group
struct SplitWalk {
  int lane_bits;  // log2 of the lanes per row
  int rows;       // rows per step
  int chunks;     // steps per row
  int per_chunk;  // (s * per_chunk) >> 16 == s / chunks for the few steps s there are
};
__host__ __device__ inline SplitWalk split_walk(int n_bins) {
  SplitWalk w;
  w.lane_bits = n_bins <= 16 ? 4 : (n_bins <= 32 ? 5 : 6);
  w.rows = 64 >> w.lane_bits;
  w.chunks = (n_bins + 63) / 64;
  w.per_chunk = 65536 / w.chunks + 1;
  return w;
}
// features per group at most: what fits the local memory budget
constexpr int kSplitMaxGroup = 16;
inline int split_max_group(int n_bins) {
  int cap = kSplitLdsBudget / split_feature_bytes(n_bins);
  if (cap > kSplitMaxGroup) cap = kSplitMaxGroup;
  const SplitWalk w = split_walk(n_bins);
  constexpr int most = kSplitSteps * (kSplitThreads / 64);
  if (cap > most / w.chunks * w.rows) cap = most / w.chunks * w.rows;
  return cap < 1 ? 1 : cap;
}
// steps a wavefront takes of a group
inline int split_steps(int n_bins, int group) {
  const SplitWalk w = split_walk(n_bins);
  return ((group + w.rows - 1) / w.rows * w.chunks + kSplitThreads / 64 - 1) / (kSplitThreads / 64);
}

// Arg-max over the threads of a workgroup under the order "larger gain, then smaller index"
// (index < 0: no candidate): exchanges inside each wavefront, then the four wavefront
// results through local memory.  The order is total, so the result does not depend on how
// the comparisons are arranged.  Every thread returns with the winner in (gain, idx).
__device__ __forceinline__ void block_argmax(double& gain, int32_t& idx, double* s_gain, int32_t* s_idx) {
  auto better = [](double g2, int32_t i2, double g1, int32_t i1) {
    return i2 >= 0 && (i1 < 0 || g2 > g1 || (g2 == g1 && i2 < i1));
  };
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const double g2 = __shfl_xor(gain, o);
    const int32_t i2 = __shfl_xor(idx, o);
    if (better(g2, i2, gain, idx)) {
      gain = g2;
      idx = i2;
    }
  }
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    s_gain[wave] = gain;
    s_idx[wave] = idx;
  }
  __syncthreads();
  gain = s_gain[0];
  idx = s_idx[0];
#pragma unroll
  for (int w = 1; w < kSplitThreads / 64; ++w) {
    const double g2 = s_gain[w];
    const int32_t i2 = s_idx[w];
    if (better(g2, i2, gain, idx)) {
      gain = g2;
      idx = i2;
    }
  }
  __syncthreads();  // the scratch may be reused
}

// Gain scan of Sec. 3.3.  A workgroup takes `passes` groups of `group` consecutive features, one
// group at a time:
//  1. Their histogram rows are copied into local memory as doubles.
//  2. One lane per (feature, statistic) runs the left-to-right prefix sum of grad, hess
//     or count in fp64, bins ascending (this fixes the rounding order).
//  3. All lanes then evaluate the gain of every (feature, threshold) pair from those
//     prefixes -- the divisions, the expensive part -- and keep the best pair under
//     the order "larger gain, then smaller feature, then smaller bin".
// Feature totals are the prefix at the last bin, right = total - left, a threshold is
// admissible when both sides hold >= 1 sample and >= min_child_hess of hessian.
// and keeps the best pair over its groups in registers.  (Requesting the rows of the next group before
// the prefix sums of the present one costs more registers than the wait is worth: 165 instead of 95, two
// workgroups per CU fewer, 64 histograms of 2,000 x 63 bins in 66 us instead of 50.)
//  4. The workgroup that finishes last for its histogram (a ticket taken after its own
//     candidate is written and fenced; nobody waits) reduces the candidates of all
//     workgroups to the histogram's split record: workgroups hold ascending feature
//     groups, so "smaller candidate index" is "smaller feature".
// grid.y = histogram of the call; histogram y starts hist_stride bins after histogram
// y - 1 (the stride may be negative: any two histograms of a pool can be searched in
// one launch).  mirror (may be NULL): a second place for the records, page-locked host
// memory that the device can write, so that a caller who must look at them on the host
// needs no copy after the kernel, only to wait for it.
// sib (sib.n may be 0): histograms sib.first .. sib.first + sib.n - 1 of the call are siblings
// by subtraction that do not exist yet: histogram sib.first + j is first formed, element by
// element as hist_subtract_kernel does it, as (pool histogram parent_slot[j]) - (histogram j of
// the call, the built child), written to its place and searched in the same pass: every
// (feature, bin) is read by exactly one workgroup, which also writes the difference.
constexpr int kSplitSiblings = 512;
struct SplitSiblings {
  const gbdt_bin_t* pool;  // histograms of hist_elems bins each
  int32_t first, n;
  int32_t parent_slot[kSplitSiblings];
};
struct NoSiblings {};  // (a launch without siblings does not carry the table)

// STEPS: register rows for the steps of a wavefront (4 or kSplitSteps; groups of few steps leave more
// workgroups room on a CU).  MANY: a launch of more workgroups than the machine holds at once, where
// workgroups per CU count more than one workgroup's time.  SIB: SplitSiblings or NoSiblings.
template <int STEPS, bool MANY, typename SIB>
__global__ void __launch_bounds__(kSplitThreads)
split_gain_kernel(gbdt_bin_t* hist, int64_t hist_stride, int32_t n_features,
                  int32_t n_bins, int32_t group, int32_t passes, double lambda, double min_child_hess,
                  SplitCand* __restrict__ cand, gbdt_split_t* __restrict__ out,
                  gbdt_split_t* __restrict__ mirror, SIB sib) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double s_gain[kSplitThreads / 64];
  __shared__ int32_t s_pair[kSplitThreads / 64];
  __shared__ int s_last;
  constexpr int kWaves = kSplitThreads / 64;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
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
  cand += (size_t)blockIdx.y * gridDim.x;
  out += blockIdx.y;
  const int B = n_bins;
  const int Bp = split_padded_bins(B);
  const int S = split_row(B);
  // layout (doubles): pg[group][S] | ph[group][S] | pn[group][S] | parent[group]
  double* pg = reinterpret_cast<double*>(smem);
  double* ph = pg + (size_t)group * S;
  double* pn = ph + (size_t)group * S;
  double* parent = pn + (size_t)group * S;

  const SplitWalk walk = split_walk(B);
  const int row_lane = lane >> walk.lane_bits;               // row of the step
  const int bin_lane = lane & ((1 << walk.lane_bits) - 1);   // bin inside the step's chunk
  // step i of this wavefront: (first row, first bin); rows are dealt over the wavefronts step by step
  auto step_at = [&](int i, int& row0, int& bin0) {
    const int s = i * kWaves + wave;
    const int r = (s * walk.per_chunk) >> 16;
    row0 = r * walk.rows;
    bin0 = (s - r * walk.chunks) * 64;
  };
  // this lane's place relative to its step's first row and bin (the rest is uniform): in a histogram, in LDS
  const uint32_t lane_bin = (uint32_t)(row_lane * B + bin_lane);
  const int lane_cell = row_lane * S + bin_lane;

  // The workgroup takes `passes` groups of `group` consecutive features one after the other and
  // keeps, per thread, the best pair seen so far with everything the record needs: one
  // candidate and one ticket per workgroup, however many features it looked at.
  const int32_t f_first = (int32_t)blockIdx.x * passes * group;
  gbdt_bin_t held[STEPS], held_parent[STEPS];
  auto request = [&](int32_t f0, int32_t nf) {
    const gbdt_bin_t* src = (is_sib ? built : hist) + (size_t)f0 * B;
    const gbdt_bin_t* src_parent = is_sib ? sib_parent + (size_t)f0 * B : nullptr;
#pragma unroll
    for (int i = 0; i < STEPS; ++i) {
      int row0, bin0;
      step_at(i, row0, bin0);
      gbdt_bin_t v = {0.0f, 0.0f, 0u}, q = {0.0f, 0.0f, 0u};
      if (row0 + row_lane < nf && bin0 + bin_lane < B) {
        v = (src + (row0 * B + bin0))[lane_bin];
        if (is_sib) q = (src_parent + (row0 * B + bin0))[lane_bin];
      }
      held[i] = v;
      held_parent[i] = q;
    }
  };
  auto features_of = [&](int32_t f0) { return n_features - f0 < group ? n_features - f0 : group; };

  double best_gain = 0.0;
  int32_t best_pair = -1;  // (feature - f_first) * (B - 1) + bin, ascending in (feature, bin)
  double best_gl = 0.0, best_hl = 0.0, best_nl = 0.0, best_g = 0.0, best_h = 0.0, best_n = 0.0;
  for (int32_t pass = 0; pass < passes; ++pass) {
    const int32_t f0 = f_first + pass * group;
    if (f0 >= n_features) break;  // (the same for every thread)
    const int32_t nf = features_of(f0);
    if (pass > 0) __syncthreads();  // the sums of the group before are no longer needed

    // 1. every bin's (gradient, hessian, count) as doubles (all exact), zeros in the padding
    request(f0, nf);
#pragma unroll
    for (int i = 0; i < STEPS; ++i) {
      int row0, bin0;
      step_at(i, row0, bin0);
      if (row0 + row_lane < nf && bin0 + bin_lane < Bp) {
        gbdt_bin_t v = held[i];
        if (is_sib) {
          v.grad = held_parent[i].grad - v.grad;
          v.hess = held_parent[i].hess - v.hess;
          v.count = held_parent[i].count - v.count;
          if (bin0 + bin_lane < B) (hist + ((size_t)f0 * B + row0 * B + bin0))[lane_bin] = v;
        }
        const int e = row0 * S + bin0 + lane_cell;
        pg[e] = (double)v.grad;
        ph[e] = (double)v.hess;
        pn[e] = (double)v.count;
      }
    }
    __syncthreads();

    // 2. running sums in place, strictly left to right, one lane per (statistic, feature).
    // The chain of dependent fp64 adds is the critical path of a lone histogram: there two
    // register blocks of kSplitBlock bins are used in turn, without copies: while one is added
    // and written back, the other one's values are on their way from local memory.
    if (tid < 3 * nf) {
      const int st = tid / nf;
      const int fl = tid - st * nf;
      double2* p = reinterpret_cast<double2*>(pg + ((size_t)st * group + fl) * S);
      constexpr int kPairs = kSplitBlock / 2;
      const int n_blocks = Bp / kSplitBlock;
      double2 va[kPairs];
#pragma unroll
      for (int i = 0; i < kPairs; ++i) va[i] = p[i];
      double acc = 0.0;
      auto add_block = [&](double2 (&v)[kPairs], int block) {
#pragma unroll
        for (int i = 0; i < kPairs; ++i) {
          v[i].x = acc + v[i].x;
          v[i].y = v[i].x + v[i].y;
          acc = v[i].y;
        }
#pragma unroll
        for (int i = 0; i < kPairs; ++i) p[block * kPairs + i] = v[i];
      };
      if constexpr (MANY) {
        for (int k = 0; k < n_blocks; ++k) {
          if (k > 0) {
#pragma unroll
            for (int i = 0; i < kPairs; ++i) va[i] = p[k * kPairs + i];
          }
          add_block(va, k);
        }
      } else {
        double2 vb[kPairs];
        for (int k = 0; k < n_blocks; k += 2) {
          const bool has_b = k + 1 < n_blocks;
          if (has_b) {
#pragma unroll
            for (int i = 0; i < kPairs; ++i) vb[i] = p[(k + 1) * kPairs + i];
          }
          add_block(va, k);
          if (k + 2 < n_blocks) {
#pragma unroll
            for (int i = 0; i < kPairs; ++i) va[i] = p[(k + 2) * kPairs + i];
          }
          if (has_b) add_block(vb, k + 1);
        }
      }
    }
    // The parent terms need sums that other lanes of the first wavefront wrote, and only those: the fences keep
    // the compiler from moving the reads up, and no other wavefront has to be waited for.
    static_assert(3 * kSplitMaxGroup <= 64, "the running sums of a group are the work of one wavefront");
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (tid < nf) {
      const double G = pg[tid * S + B - 1], H = ph[tid * S + B - 1];
      parent[tid] = __ddiv_rn(__dmul_rn(G, G), H + lambda);
    }
    __syncthreads();

    // 3. the gains of this group's (feature, threshold) pairs
#pragma unroll 1
    for (int i = 0; i < STEPS; ++i) {
      int row0, bin0;
      step_at(i, row0, bin0);
      if (row0 >= nf) break;  // (the same for the whole wavefront)
      const int fl = row0 + row_lane, t = bin0 + bin_lane;
      if (fl >= nf || t >= B - 1) continue;
      const int e = row0 * S + bin0 + lane_cell, last = fl * S + B - 1;
      const double GL = pg[e], HL = ph[e], NL = pn[e];
      const double G = pg[last], H = ph[last], N = pn[last];
      const double GR = G - GL, HR = H - HL;
      const double NR = N - NL;  // counts are exact in fp64
      const bool ok = NL >= 1.0 && NR >= 1.0 && HL >= min_child_hess && HR >= min_child_hess;
      if (ok) {
        const double lt = __ddiv_rn(__dmul_rn(GL, GL), HL + lambda);
        const double rt = __ddiv_rn(__dmul_rn(GR, GR), HR + lambda);
        const double gain = __dsub_rn(__dadd_rn(lt, rt), parent[fl]);
        if (best_pair < 0 || gain > best_gain) {  // pairs ascend: ties keep the earlier pair
          best_gain = gain;
          best_pair = (f0 - f_first + fl) * (B - 1) + t;
          best_gl = GL;
          best_hl = HL;
          best_nl = NL;
          best_g = G;
          best_h = H;
          best_n = N;
        }
      }
    }
  }
  const int32_t my_pair = best_pair;
  block_argmax(best_gain, best_pair, s_gain, s_pair);
  // the thread that holds the winning pair (thread 0 when there is none) hands the candidate over
  const bool writer = best_pair < 0 ? tid == 0 : my_pair == best_pair;
  if (writer) {
    SplitCand c;
    const int32_t e = best_pair;
    if (e < 0) {
      c.gain = 0.0;
      c.gl = c.hl = c.gr = c.hr = 0.0;
      c.nl = c.nr = 0;
      c.feature = -1;
      c.bin = -1;
    } else {
      const int fl = e / (B - 1);
      const int t = e - fl * (B - 1);
      c.gain = best_gain;
      c.gl = best_gl;
      c.hl = best_hl;
      c.nl = (uint32_t)best_nl;
      c.gr = best_g - best_gl;
      c.hr = best_h - best_hl;
      c.nr = (uint32_t)(best_n - best_nl);
      c.feature = f_first + fl;
      c.bin = t;
    }
    store_cand(cand + blockIdx.x, c);
    // HARDWARE ASSUMPTION (gfx942 / gfx950, not the language's memory model): a device-scope
    // atomic store is written through to the point where the other XCDs' device-scope atomic
    // loads read it, and is acknowledged (vmcnt) only then.  Waiting for the candidate's
    // stores (vmcnt(0)) before taking the ticket is therefore all the release this hand-off
    // needs, and the reader needs no acquire because it reads the candidates with device-scope
    // atomic loads only.  A release / acquire pair in the language's sense would also write back
    // and invalidate every line of the L2, which costs tens of microseconds here -- several
    // times the whole kernel.  tests/test_gpu_robustness.py runs 64 x 250 workgroups of this
    // hand-off 20 times and every split test goes through it; on a part where the assumption
    // did not hold those tests would show stale candidates.
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0); expcnt, lgkmcnt untouched
    unsigned int* ticket = split_ticket(blockIdx.y);
    const unsigned int old = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool last = old == gridDim.x - 1;
    if (last)  // back to zero for the next launch
      __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_last = last;
  }
  __syncthreads();
  if (!s_last) return;
  // The ticket's value has arrived, so every other workgroup's candidate was acknowledged
  // before its ticket; the loads below are device-scope atomics and bypass stale caches.

  // ---- the histogram's last workgroup: arg-max over all candidates.  Each thread folds
  // a strided subset in ascending order, then a tree reduction.
  // (Two round trips to the other workgroups' results: the keys of all candidates, then the winner's record,
  // which its owner fetches and writes.  Fetching whole candidates at once saves the second, but 56 bytes
  // apart seven words of each take longer than that: a lone histogram of 500 x 64, 250 candidates, 9.9 us so
  // and 9.5 with keys first; 28 candidates 6.9 either way.)
  const int32_t n_cand = (int32_t)gridDim.x;
  double bg = 0.0;
  int32_t bi = -1;
  for (int32_t i = tid; i < n_cand; i += kSplitThreads) {
    double gain;
    int32_t feature;
    load_cand_key(cand + i, &gain, &feature);
    if (feature >= 0 && (bi < 0 || gain > bg)) {  // i ascends, so ties keep the smaller feature
      bg = gain;
      bi = i;
    }
  }
  const int32_t my_cand = bi;
  block_argmax(bg, bi, s_gain, s_pair);
  if (bi < 0 ? tid == 0 : my_cand == bi) {
    gbdt_split_t r;
    if (bi < 0) {
      r.feature = -1;
      r.bin = -1;
      r.gain = 0.0f;
      r.left_grad = r.left_hess = r.right_grad = r.right_hess = 0.0f;
      r.left_count = r.right_count = 0;
    } else {
      const SplitCand mine = load_cand(cand + bi);
      r.feature = mine.feature;
      r.bin = mine.bin;
      r.gain = (float)mine.gain;
      r.left_grad = (float)mine.gl;
      r.left_hess = (float)mine.hl;
      r.left_count = mine.nl;
      r.right_grad = (float)mine.gr;
      r.right_hess = (float)mine.hr;
      r.right_count = mine.nr;
    }
    *out = r;
    if (mirror) mirror[blockIdx.y] = r;
  }
}

}  // namespace

#endif  // GBDT_SPLIT_KERNELS_H_
