// Window calibration with Section 2, step (2) of the paper read literally (the band mask mode):
// the attention map of query scale k is cut into parts -- the first three key scales together,
// then one part per key scale -- and in every part the window is the band of radius r around
// the part's diagonal, floor((2 i + 1) n / (2 s_k^2)) at query i of a part of n columns; the
// band grows from radius zero until it holds the fraction R_0 of the part's values.
//
// The sums of a part's values by distance from the diagonal come from the streaming pass of
// calib_stream.h (a part's columns are consecutive tokens); a second, small kernel adds the row
// shares of a part in a fixed order, forms the in-band sums by prefix and picks the radius.
#include "calib_stream.h"

#include <cstring>

namespace lv {

namespace {

constexpr int kBandThreads = 256;
// Row shares of a part: sixteen at most, up to 31 where a share keeps 64 rows (more shares of fewer rows cost
// more than they spread: eight scales of side 24, 36 / 19 rows: 84 / 115 us).  One scale of side 64, four samples,
// sixteen / 31 shares: 945 / 596 us; scales 1 to 64, 3 samples x 2 heads: 1172 / 705.  The workspace stays
// below twice sixteen offsets per column.
inline int band_row_shares(int rows) { return rows / 64 <= 16 ? 16 : rows / 64 < 31 ? rows / 64 : 31; }
constexpr int kMaxPartCols = 4096;    // per-distance sums of a part live in LDS in the pick kernel

struct BandArgs {
  StreamGeom g;
  int n_parts, mcols;
  int64_t head_stride;             // doubles of partial sums per head
  int64_t base[kMaxScales];        // query scale k's [row shares][off[k + 1]] sums inside a head's region, by
                                   // the part's first token + distance
  double* partial;
  int32_t* radius;      // [H][K][K]
  double* mass;         // [H][K][K][mcols] or nullptr
  double r0;
};

__host__ __device__ inline int parts_of(int k) { return k < kMergedScales ? 1 : k - kMergedScales + 2; }

// part of query scale k that key scale j belongs to: its first and last key scale
__host__ __device__ inline int part_first(int j) { return j < kMergedScales ? 0 : j; }
__host__ __device__ inline int part_last(int k, int j) {
  return j >= kMergedScales ? j : k < kMergedScales - 1 ? k : kMergedScales - 1;
}

struct BandWalk {
  static constexpr int kClasses = 2;     // 1: the column wrapped (offset u - n)
  const StreamGeom& g; const StreamTask& t;
  int n, u, row, drow, tok0;
  unsigned q, rem, dq, dr, den;          // the diagonal at `row` = q, exactly: (2 row + 1) n = q den + rem, den = 2 s_k^2
  __device__ void start(int e, int row0, int step) {
    int j = t.ja;
    while (j + 1 < t.jb && t.col0 + e >= g.off[j + 1]) ++j;
    tok0 = g.off[part_first(j)];
    n = g.off[part_last(t.k, j) + 1] - tok0;
    u = t.col0 + e - tok0;
    row = row0; drow = step;
    // (sides are at most 64 and a part has at most 4096 columns: all products stay below 2^26)
    den = 2u * (unsigned)(g.s[t.k] * g.s[t.k]);
    const unsigned num = (2u * (unsigned)row0 + 1u) * (unsigned)n, dnum = 2u * (unsigned)step * (unsigned)n;
    q = num / den; rem = num - q * den;
    dq = dnum / den; dr = dnum - dq * den;
  }
  __device__ int64_t next(int& cls) {
    int c = (int)q + u;
    cls = c >= n;
    c -= cls ? n : 0;
    const int64_t at = (int64_t)row * g.L + tok0 + c;
    row += drow; q += dq; rem += dr;
    if (rem >= den) { rem -= den; ++q; }
    return at;
  }
};

// grid (heads, slots), the slots with the most work first.
// Measured (8 samples x 30 heads x 680^2): 56 us, 4.9 TB/s of the block-causal values; the former
// kernel, one lane per signed offset (half of them idle in any row) and one load at a time, took 243 us.
// k_band_pick: 12 us; 14.5 with LDS for the widest part that there can be (four workgroups per CU, two rounds of
// them), 46 with one thread for the prefix and the 64-bit divisions.
template <int NB>
__global__ __launch_bounds__(kStreamThreads) void k_band_stream(BandArgs a) {
  extern __shared__ __align__(16) unsigned char band_smem[];
  const StreamGeom& g = a.g;
  const StreamTask t = stream_task(g);
  double* const acc = (double*)band_smem;                                      // [2][entries]
  BandWalk walk{g, t};
  stream_sums<NB>(g, t, walk, acc);
  __syncthreads();
  const int R = stream_rows_at_once(t);
  double* out = a.partial + (int64_t)t.h * a.head_stride + a.base[t.k] + (int64_t)t.split * g.off[t.k + 1] + t.col0;
  for (int e = threadIdx.x; e < t.ncols; e += kStreamThreads) {
    int j = t.ja;
    while (j + 1 < t.jb && t.col0 + e >= g.off[j + 1]) ++j;
    const int tok0 = g.off[part_first(j)], p0 = tok0 - t.col0, n = g.off[part_last(t.k, j) + 1] - tok0, d = e - p0;
    double v = 0.0;
    for (int r = 0; r < R; ++r) {
      const double* s = acc + (R > 1 ? r * t.ncols : 0) + p0;
      v += s[d];
      if (d > 0) v += s[g.entries + n - d];
    }
    out[e] = v;
  }
}

// grid (parts, heads): per-distance sums of the part, prefix, radius
__global__ __launch_bounds__(kBandThreads) void k_band_pick(BandArgs a) {
  extern __shared__ __align__(16) unsigned char band_smem[];
  double* const by_dist = (double*)band_smem;                    // [a.mcols]
  double* const carry = by_dist + a.mcols;
  __shared__ int found_at;
  const StreamGeom& g = a.g;
  const int h = blockIdx.y, K = g.K;
  int k = 0, pt = blockIdx.x;                                    // parts of query scale 0, then of query scale 1, ...
  while (pt >= parts_of(k)) { pt -= parts_of(k); ++k; }
  const int first = pt == 0 ? 0 : pt + kMergedScales - 1, last = part_last(k, first);
  const int tok0 = g.off[first], n = g.off[last + 1] - tok0;
  const double* part = a.partial + (int64_t)h * a.head_stride + a.base[k] + tok0;
  for (int d = threadIdx.x; d < n; d += kBandThreads) by_dist[d] = sum_partials(part + d, g.splits[k], g.off[k + 1]);
  const int found = prefix_and_pick(by_dist, n, a.r0, carry, &found_at);   // the band grows from zero
  if (threadIdx.x == 0) {
    int32_t* rad = a.radius + ((int64_t)h * K + k) * K;
    for (int j = first; j <= last; ++j) rad[j] = found;
    if (first == 0)                                              // the first part also marks the key scales above k
      for (int j = k + 1; j < K; ++j) rad[j] = -1;
  }
  if (a.mass) {
    for (int j = 0; j < K; ++j) {
      double* m = a.mass + (((int64_t)h * K + k) * K + j) * a.mcols;
      if (j >= first && j <= last) {
        for (int r = threadIdx.x; r < a.mcols; r += kBandThreads) m[r] = by_dist[r < n ? r : n - 1];
      } else if (first == 0 && j > k) {
        for (int r = threadIdx.x; r < a.mcols; r += kBandThreads) m[r] = 0.0;
      }
    }
  }
}

litevar_status band_geom(const int32_t* scales, int32_t n_scales, int32_t H, BandArgs& a) {
  if (!scales) return fail(LITEVAR_E_INVALID_ARG, "scales is NULL");
  if (n_scales < 1 || n_scales > kMaxScales)
    return fail(LITEVAR_E_INVALID_ARG, "n_scales must be in 1..%d (got %d)", kMaxScales, n_scales);
  if (H < 1 || H > 65535) return fail(LITEVAR_E_INVALID_ARG, "H must be in 1..65535 (got %d)", H);
  std::memset(&a, 0, sizeof a);
  StreamGeom& g = a.g;
  g.K = n_scales; g.H = H;
  int64_t L = 0;
  for (int k = 0; k < n_scales; ++k) {
    if (scales[k] < 1 || scales[k] > kStreamMaxSide)
      return fail(LITEVAR_E_UNSUPPORTED, "band calibration takes scale sides 1..64 (got %d)", scales[k]);
    g.s[k] = scales[k]; g.off[k] = (int)L;
    L += (int64_t)scales[k] * scales[k];
  }
  g.off[n_scales] = (int)L;
  g.L = L;
  for (int k = 0; k < n_scales; ++k) {
    a.n_parts += parts_of(k);
    for (int j = 0; j <= k; ++j) {
      const int n = g.off[part_last(k, j) + 1] - g.off[part_first(j)];
      if (n > kMaxPartCols) return fail(LITEVAR_E_UNSUPPORTED, "a part of %d columns (at most %d)", n, kMaxPartCols);
      if (n > a.mcols) a.mcols = n;
    }
  }
  stream_plan(g, kMergedScales, [&](int k) { return band_row_shares(g.s[k] * g.s[k]); });
  int64_t stride = 0;
  for (int k = 0; k < n_scales; ++k) {
    a.base[k] = stride;
    stride += (int64_t)g.splits[k] * g.off[k + 1];
  }
  a.head_stride = stride;
  return LITEVAR_OK;
}

}  // namespace

}  // namespace lv

using namespace lv;

extern "C" {

litevar_status litevar_window_calibrate_band_workspace_bytes(const int32_t* scales, int32_t n_scales, int32_t H,
                                                             size_t* out_bytes) {
  if (!out_bytes) return fail(LITEVAR_E_INVALID_ARG, "out_bytes is NULL");
  BandArgs a;
  if (litevar_status s = band_geom(scales, n_scales, H, a)) return s;
  *out_bytes = (size_t)a.head_stride * (size_t)H * sizeof(double);
  return LITEVAR_OK;
}

litevar_status litevar_window_calibrate_band(const int32_t* scales, int32_t n_scales, const float* d_attn, int32_t N,
                                             int32_t H, float r0, void* d_workspace, size_t workspace_bytes,
                                             int32_t* d_radius, double* d_mass, void* stream) {
  BandArgs a;
  if (litevar_status s = band_geom(scales, n_scales, H, a)) return s;
  if (N < 1) return fail(LITEVAR_E_INVALID_ARG, "N must be positive");
  if (!(r0 > 0.f) || r0 > 1.f) return fail(LITEVAR_E_INVALID_ARG, "r0 must be in (0, 1] (got %g)", r0);
  if (!d_attn || !d_radius || !d_workspace) return fail(LITEVAR_E_INVALID_ARG, "d_attn, d_radius or d_workspace is NULL");
  if (((uintptr_t)d_workspace & 7) || (d_mass && ((uintptr_t)d_mass & 7)))
    return fail(LITEVAR_E_INVALID_ARG, "d_workspace and d_mass must be 8-byte aligned");
  const size_t need = (size_t)a.head_stride * (size_t)H * sizeof(double);
  if (workspace_bytes < need) return fail(LITEVAR_E_INVALID_ARG, "workspace of %zu bytes, %zu needed", workspace_bytes, need);
  a.g.N = N; a.g.p = d_attn; a.partial = (double*)d_workspace; a.radius = d_radius; a.mass = d_mass; a.r0 = (double)r0;
  hipStream_t st = (hipStream_t)stream;
  const size_t lds = (size_t)2 * a.g.entries * sizeof(double);
  const auto kernel = stream_pick(N, k_band_stream<1>, k_band_stream<2>, k_band_stream<4>, k_band_stream<8>);
  if (lds > 64 * 1024)       // (beyond the default limit of dynamically sized LDS; no allocation involved)
    if (litevar_status s = hip_check(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                         (int)lds), "hipFuncSetAttribute")) return s;
  hipLaunchKernelGGL(kernel, dim3(H, a.g.slot_begin[a.g.K]), dim3(kStreamThreads), lds, st, a);
  if (litevar_status s = hip_check(hipGetLastError(), "band calibration mass launch")) return s;
  const size_t pick_lds = (size_t)(a.mcols + a.mcols / kPrefixRun + 1) * sizeof(double);   // (at most 34.8 KB)
  hipLaunchKernelGGL(k_band_pick, dim3(a.n_parts, H), dim3(kBandThreads), pick_lds, st, a);
  return hip_check(hipGetLastError(), "band calibration pick launch");
}

}  // extern "C"
