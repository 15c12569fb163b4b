// The streaming pass of both window calibrations (calibrate.hip: square windows, calibrate_band.hip:
// bands): sums of a part's values by distance from the row's centre, for scale sides up to 64.
//
// A value's distance depends on its offset from the centre of its map row.  A workgroup owns a
// share of the rows of one query scale and one SEGMENT of key columns: consecutive whole parts
// that together have at most 256 columns, or one larger part.  A lane owns one offset class of a
// part of n columns: in a row with centre c it reads column (c + u) mod n, i.e. offset u, or
// u - n where the column wraps around.  So every lane reads exactly one value per row (a plain
// lane-per-offset walk would leave half of them idle), the lanes of a wave read a permutation of
// consecutive columns, and the sums stay in registers: one fp64 sum per wrap state (two for a
// band, 2 x 2 for a square window).  The samples of a row share its centre and are added first.
// Narrow segments put several rows side by side in the workgroup.  At the end the sums go through
// LDS once and are folded by distance in a fixed order: no atomics, two launches give the same bits.
//
// Bound: the map's values, 4 bytes each, read once.  Measured (8 samples x 30 heads x 680^2, 275 MB
// of block-causal values; a large copy reaches 5.3 TB/s): sixteen loads in flight per lane 63 / 56 us
// (window / band), eight 67 / 59 us; 32 rows per workgroup instead of 16: 64 / 58 us.
#pragma once
#include "internal.h"

namespace lv {

constexpr int kStreamThreads = 256;
constexpr int kStreamMaxSide = 64;
constexpr int kStreamLoads = 16;         // loads in flight per lane: samples of one row, or of several rows
constexpr int kStreamRowsAtOnce = 32;    // rows side by side in a workgroup at most (they are folded serially)
constexpr int kStreamRowsPerBlock = 16;  // rows of a query scale per workgroup, where the workspace has room:
                                         // 16 x 256 columns x 8 samples are 131 KB, a few microseconds

struct StreamGeom {
  int K, N, H;
  int entries;                           // columns of the widest segment, at least kStreamThreads
  int s[kMaxScales], off[kMaxScales + 1];
  int64_t L;
  int slot_begin[kMaxScales + 1];        // workgroups (of one head) ahead of launch entry i, which is query
                                         // scale K - 1 - i: the scales with the most work start first
  int splits[kMaxScales];                // row shares of a query scale
  uint8_t seg_first[kMaxScales + 1];     // first key scale of every segment
  const float* p;                        // [N][H][L][L]
};

// K, s, off, L are set; lead: how many key scales the first part spans; max_splits(k): row shares that
// the workspace has room for
template <class MaxSplits>
inline void stream_plan(StreamGeom& g, int lead, MaxSplits max_splits) {
  int n_seg = 0;
  g.entries = kStreamThreads;
  for (int j = 0; j < g.K;) {
    int e = j + (j == 0 ? (lead < g.K ? lead : g.K) : 1);
    while (e < g.K && g.off[e + 1] - g.off[j] <= kStreamThreads) ++e;
    g.seg_first[n_seg++] = (uint8_t)j;
    if (g.off[e] - g.off[j] > g.entries) g.entries = g.off[e] - g.off[j];
    j = e;
  }
  g.seg_first[n_seg] = (uint8_t)g.K;
  int at = 0;
  for (int i = 0; i < g.K; ++i) {
    const int k = g.K - 1 - i, nk = g.s[k] * g.s[k], cap = max_splits(k);
    const int want = (nk + kStreamRowsPerBlock - 1) / kStreamRowsPerBlock;
    g.splits[k] = want < cap ? want : cap;
    int segs = 0;
    while (segs < n_seg && g.seg_first[segs] <= k) ++segs;
    g.slot_begin[i] = at;
    at += g.splits[k] * segs;
  }
  g.slot_begin[g.K] = at;
}

struct StreamTask { int h, k, ja, jb, split, i0, i1, col0, ncols; };   // key scales [ja, jb), rows [i0, i1)

// (grid (heads, slots): a one-dimensional one would pass 2^32 threads, where launches wrap without an
// error, at 65 535 heads and 256 slots; workgroups start in the order of x)
__device__ inline StreamTask stream_task(const StreamGeom& g) {
  StreamTask t;
  const int slot = (int)blockIdx.y;
  t.h = (int)blockIdx.x;
  const int lane = threadIdx.x & 63;
  const bool started = lane < g.K && g.slot_begin[min(lane, g.K)] <= slot;
  const int i = __builtin_amdgcn_readfirstlane(__builtin_popcountll(__ballot(started)) - 1);
  t.k = g.K - 1 - i;
  const int S = g.splits[t.k], local = slot - g.slot_begin[i], seg = local / S;
  t.split = local - seg * S;
  t.ja = g.seg_first[seg];
  t.jb = min((int)g.seg_first[seg + 1], t.k + 1);
  t.col0 = g.off[t.ja]; t.ncols = g.off[t.jb] - t.col0;
  const int nk = g.s[t.k] * g.s[t.k], rows = (nk + S - 1) / S;
  t.i0 = t.split * rows; t.i1 = min(nk, t.i0 + rows);
  return t;
}

// rows that a workgroup walks side by side (no more than it has: they are folded one after the other)
__device__ inline int stream_rows_at_once(const StreamTask& t) {
  return t.ncols > kStreamThreads / 2 ? 1 : max(1, min(min(kStreamThreads / t.ncols, kStreamRowsAtOnce), t.i1 - t.i0));
}

// Fills acc[class][row at once x column] (pitch g.entries) with the sums of the task's values.
// Walk: walk.start(column, row, step) places the lane on a column of the segment and its first row;
// walk.next(cls) returns the element offset of the lane's value in the map of (sample 0, head),
// relative to query scale k's first row, and its class, and moves on by `step` rows.
// NB samples of kStreamLoads / NB rows are in flight at a time.
template <int NB, class Walk>
__device__ inline void stream_sums(const StreamGeom& g, const StreamTask& t, Walk& walk, double* acc) {
  constexpr int RB = kStreamLoads / NB, NC = Walk::kClasses;
  const int R = stream_rows_at_once(t);
  const float* base = g.p + ((int64_t)t.h * g.L + g.off[t.k]) * g.L;
  const int64_t sample = (int64_t)g.H * g.L * g.L;
  for (int e0 = 0; e0 < t.ncols; e0 += kStreamThreads) {
    const int r = R > 1 ? (int)threadIdx.x / t.ncols : 0;
    const int e = R > 1 ? (int)threadIdx.x - r * t.ncols : e0 + (int)threadIdx.x;
    if (r >= R || e >= t.ncols) continue;
    double sum[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) sum[c] = 0.0;
    walk.start(e, t.i0 + r, R);
    for (int i = t.i0 + r; i < t.i1; i += R * RB) {
      const float* src[RB];
      int cls[RB];
#pragma unroll
      for (int b = 0; b < RB; ++b) {
        // (a row past the share's end: the first one is read again and not added)
        const bool in = i + b * R < t.i1;
        int c = 0;
        const int64_t at = in ? walk.next(c) : 0;
        src[b] = in ? base + at : src[0];
        cls[b] = in ? c : -1;
      }
      double x[RB];
#pragma unroll
      for (int b = 0; b < RB; ++b) x[b] = 0.0;
      for (int n0 = 0; n0 < g.N; n0 += NB) {
        float v[RB][NB];
#pragma unroll
        for (int b = 0; b < RB; ++b)
#pragma unroll
          for (int m = 0; m < NB; ++m) v[b][m] = src[b][min(n0 + m, g.N - 1) * sample];
#pragma unroll
        for (int b = 0; b < RB; ++b)
#pragma unroll
          for (int m = 0; m < NB; ++m) x[b] += n0 + m < g.N ? (double)v[b][m] : 0.0;
      }
#pragma unroll
      for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int c = 0; c < NC; ++c) sum[c] += cls[b] == c ? x[b] : 0.0;
    }
    const int at = R > 1 ? (int)threadIdx.x : e;
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c * g.entries + at] = sum[c];
  }
}

// samples of a row in flight together: the instantiation for N samples
template <class F1, class F2, class F4, class F8>
inline auto stream_pick(int N, F1 f1, F2 f2, F4 f4, F8 f8) { return N >= 5 ? f8 : N >= 3 ? f4 : N == 2 ? f2 : f1; }

// Sum of `count` partial sums `stride` values apart, in order, sixteen loads in flight (a row share
// past the last is read again and not added).  Each round is a trip to memory: the partial sums come
// from other XCDs.
__device__ inline double sum_partials(const double* p, int count, int64_t stride) {
  constexpr int kInFlight = 16;
  double sum = 0.0;
  for (int i = 0; i < count; i += kInFlight) {
    double v[kInFlight];
#pragma unroll
    for (int u = 0; u < kInFlight; ++u) v[u] = p[min(i + u, count - 1) * stride];
#pragma unroll
    for (int u = 0; u < kInFlight; ++u) sum += i + u < count ? v[u] : 0.0;
  }
  return sum;
}

// val[0 .. n) (LDS, sums by distance) becomes its prefix sums; returns the smallest d with val[d] >= r0
// of the total, n - 1 if there is none.  All threads of the workgroup call it, carry: n / kPrefixRun + 1
// words.  Runs of kPrefixRun values are added in order side by side, then their totals in order, so
// that the sums never fall and a run of zeros adds nothing.  (One thread's chain over all values is an
// LDS round trip for every sixteen of them: band calibrations of one scale of side 64 took 342 us, 285
// like this; side 48 163 and 130; 30 heads of sides up to 16, 8 samples 66.1 and 63.3.  The ratio is a
// 64-bit division, by all threads at once.)
constexpr int kPrefixRun = 16;
__device__ inline int prefix_and_pick(double* val, int n, double r0, double* carry, int* found) {
  __syncthreads();
  const int runs = (n + kPrefixRun - 1) / kPrefixRun;
  for (int b = threadIdx.x; b < runs; b += blockDim.x) {
    double v[kPrefixRun];
#pragma unroll
    for (int u = 0; u < kPrefixRun; ++u) v[u] = val[min(b * kPrefixRun + u, n - 1)];
    double in = 0.0;
#pragma unroll
    for (int u = 0; u < kPrefixRun; ++u) {
      in += v[u];
      if (b * kPrefixRun + u < n) val[b * kPrefixRun + u] = in;
    }
  }
  if (threadIdx.x == 0) *found = n - 1;
  __syncthreads();
  if (runs > 1) {
    if (threadIdx.x == 0) {
      double in = 0.0;
      for (int b0 = 0; b0 < runs - 1; b0 += kPrefixRun) {
        double v[kPrefixRun];
#pragma unroll
        for (int u = 0; u < kPrefixRun; ++u) v[u] = val[min((b0 + u + 1) * kPrefixRun, n) - 1];
#pragma unroll
        for (int u = 0; u < kPrefixRun; ++u) {
          in += v[u];
          if (b0 + u < runs - 1) carry[b0 + u] = in;
        }
      }
    }
    __syncthreads();
    for (int d = kPrefixRun + threadIdx.x; d < n; d += blockDim.x) val[d] += carry[d / kPrefixRun - 1];
    __syncthreads();
  }
  const double total = val[n - 1];
  int mine = n - 1;
  for (int d = threadIdx.x; d < n; d += blockDim.x)
    if (total == 0.0 || val[d] / total >= r0) { mine = d; break; }
  atomicMin(found, mine);
  __syncthreads();
  return *found;
}

}  // namespace lv
