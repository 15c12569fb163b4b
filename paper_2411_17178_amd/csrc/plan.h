// Internal layout of a LiteVAR windowed-attention plan and the integer geometry
// shared by the host sizing pass and the device builder kernels.
//
// Vocabulary (Section 2 of the paper for scales/parts/windows; the tiling is ours):
//   patch   16 queries of one scale = the 16 columns of one MFMA tile, handled by one
//           64-lane wave: a 4x4 block of the scale's grid (window mode) or 16 consecutive
//           queries (band mode);
//   group   up to NW patches of one query scale handled by one workgroup that
//           stages the keys they need through an LDS ring;
//   union   the group's key list: for every part of the attention map the keys that any of
//           its queries keeps (window mode: the bounding box of the windows in every key
//           scale, row-major; band mode: one column range per part), parts in ascending order;
//   step    32 keys of one patch's own key list (two 16-key MFMA tiles for
//           K Q^T, one K=32 MFMA slice for V^T P^T) with one mask bit per
//           (query, key);
//   phase   the group processes the union list in chunks of C keys; a step is
//           run in the phase of its last key and may reach back A chunks;
//   head group   heads that share one radius table share one set of groups, lists and steps;
//   wide patch   32 queries of one scale = the 32 columns of one 32x32 MFMA tile.  The groups of 16 patches
//           carry a second work-list over the same key list: up to eight wide patches (4 x 8
//           queries, or what covers the group's queries with the fewest key rows; band mode: 32
//           consecutive queries) with steps of 32 keys of their own.  The 16-patch kernel's eight-wave form
//           walks it, and the list's order, the phase tables and the ring offsets of the steps are theirs; of the patches of
//           16 such plans hold tokens and masks only, which the exports, the fp32 kernel and attend_row read.  Plans that ask for the sixteen-wave
//           form (patches_per_wave = 1) have none, nor have plans one of whose wide patches would need more
//           than 65535 steps: their box can be larger than those of its two patches of 16.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <vector>

#define LV_HD __host__ __device__ inline

namespace lv {

constexpr int kMaxScales = 32;
constexpr int kMaxSide = 1024;
constexpr int kMaxRadius = 32767;    // radii are stored as int16 (band mode counts columns of a part)
constexpr int kMaxHeads = 256;       // heads with their own radius table
constexpr int kStepKeys = 32;
constexpr int kPatch = 4;
constexpr int kPatchQueries = 16;
constexpr int kWidePatches = 8;      // wide patches of a group (plans with 16 patches per group)
constexpr int kWideQueries = 32;
constexpr int kWideDesc = 16;        // bytes of a wide step's descriptor per lane
constexpr int kMergedScales = 3;     // band mode: the first part spans the first three scales
constexpr uint64_t kMagic = 0x4c56415257494e32ull;  // "LVARWIN2"

enum MaskMode { kModeWindow = 0, kModeBand = 1 };

struct Geom {
  int K, qb, qe, n_sink;
  int L, Lq, q0, smax;
  int NW;               // patches per group
  int n_wide;           // wide patches per group: kWidePatches, or 0 where the plan has none
  short grh[kMaxScales], grw[kMaxScales];   // window mode: group shape in patches (grh x grw <= NW) of every query scale
  short wph[kMaxScales], wpw[kMaxScales];   // window mode, NW = 16: queries of a wide patch of every query scale
  int C, NR, A, D;      // chunk keys (a power of two), ring depth in chunks, look-back and
                        // prefetch depth in chunks; NR = A + 1 + D
  int logC;
  int logS;             // a step spans at most A + 1 consecutive blocks of 2^logS keys (logS <= logC)
  int R;                // ring slots
  int n_groups, n_patches;   // per head group
  int mode;             // MaskMode
  int n_hg;             // head groups (1 unless the plan has one radius table per head)
  int s[kMaxScales];
  int off[kMaxScales + 1];
  int grp_off[kMaxScales + 1];  // groups are ordered by DESCENDING query scale:
                                // slot i holds scale qe-1-i; grp_off is its prefix sum
};

// The host's geometry, with the radii of ONE head group, [query scale][key scale] (Section 2, step (3): one window
// size per scale and part); < 0: dense part.  The host sizes one head group at a time; the device kernels get
// the Geom alone (2 KB less of kernel arguments in every launch) and read the tables in the blob.
struct HostGeom : Geom {
  short rad[kMaxScales][kMaxScales];
};

struct GroupDesc {   // 32 bytes
  int32_t union_base;  // first entry in union_tok
  int32_t n_union;     // real keys
  int32_t n_phases;    // ceil(n_union / C), >= 1
  int32_t k;           // query scale
  int32_t gy, gx;      // group position in units of groups (band mode: gy = index in the scale, gx = 0)
  int32_t phase_base;  // first entry in phase_end (walked_patches * n_phases int32 entries, wave-major)
  int32_t ident;       // union entries [0, ident) hold token i at position i
};

struct WaveDesc {    // 32 bytes
  int32_t step_begin;
  int32_t n_steps;
  int32_t q_base;      // local query row of the patch's first query
  int16_t sk;          // query n of the patch is row q_base + (n / 4) * sk + n % 4
  int16_t ny, nx;      // valid extent of the patch (0 = idle wave); band mode: (1, number of queries)
  int16_t kq;          // query scale index
  int32_t pairs;       // kept pairs of this patch (statistics)
  uint32_t valid;      // bit n set: column n of the patch holds a query
  uint32_t first_ends; // phase_end[0] | phase_end[min(2, n_phases - 1)] << 16: the step counts that the
                       // 16-patch kernel needs before it can start, next to the patch's other words
};
// (Wide patches use the same words: their query n is row q_base + (n / nx) * sk + n % nx, nx being the
// patch's own extent, and `pairs` holds ceil(65536 / nx), with which n / nx is one multiplication.)
static_assert(sizeof(WaveDesc) == 32 && sizeof(GroupDesc) == 32, "descriptor size");

struct Header {      // first 256 bytes of the blob
  uint64_t magic;
  uint64_t blob_bytes;
  int32_t n_groups, n_waves;
  int64_t n_steps, n_union, n_phase_entries;
  int64_t retained_pairs;
  int32_t error;       // kErrBuilder: set by the builder when the device's walk and the host's counts differ
                       // (the work-list sections are then not written beyond the counts and no kernel
                       // uses the plan);
                       // kErrWaitGaveUp: an attention kernel's bounded wait on an LDS flag ran out;
                       // kErrBounds: a kernel of the bounds-checking build found a token, a query
                       // row or an LDS offset out of range (it used index 0 instead)
  int32_t pad0;
  int64_t n_wide_steps;  // steps of the wide patches, 0 without them
  uint64_t pad[23];
};
static_assert(sizeof(Header) == 256, "header size");

enum HeaderError { kErrNone = 0, kErrBuilder = 1, kErrWaitGaveUp = 2, kErrBounds = 3 };
constexpr int kDefaultSpinLimit = 1 << 22;   // polls of about 64 cycles each

enum Section { kSecHeader = 0, kSecWin, kSecRad, kSecHeadMap, kSecGroups, kSecWaves, kSecPhaseEnd,
               kSecUnion, kSecStepAddr, kSecStepMask, kSecStepTok, kSecEnd, kNumSections };

// LDS ring geometry of the bf16 kernel: one 128-byte row per key in each of the K and V
// rings; the 16-byte piece c of the row in slot s is stored at piece position
// c ^ swizzle(s).
constexpr int kRingRowBytes = 128;
LV_HD unsigned ring_swizzle(unsigned slot) { return (slot ^ (slot >> 3)) & 7u; }

// ---- window definition (window mode) -------------------------------------------
// Inclusive interval of key coordinates of scale j kept along one axis by query
// coordinate c of scale k: centre = floor((2c+1) s_j / (2 s_k)), radius r, clipped.
struct Interval { int lo, hi; };   // empty when hi < lo

LV_HD Interval window_interval(int sk, int sj, int c, int rad) {
  Interval iv;
  if (rad < 0) { iv.lo = 0; iv.hi = sj - 1; return iv; }
  // (sides are at most kMaxSide = 1024, so the product fits 32 bits: a 64-bit division would
  // cost an order of magnitude more on the device)
  const int ctr = (int)((unsigned)((2 * c + 1) * sj) / (unsigned)(2 * sk));
  iv.lo = ctr - rad < 0 ? 0 : ctr - rad;
  iv.hi = ctr + rad > sj - 1 ? sj - 1 : ctr + rad;
  return iv;
}
inline Interval win_interval(const HostGeom& g, int k, int j, int c) {
  return window_interval(g.s[k], g.s[j], c, j < g.n_sink ? -1 : g.rad[k][j]);
}

// The builder's kernels take their intervals from the device table, which k_tables fills.
struct TableWin {        // win[((k * K + j) * smax + c) * 2 + {0, 1}] of one head group
  const int16_t* win; int K, smax;
  LV_HD Interval operator()(int k, int j, int c) const {
    const int16_t* p = win + ((size_t)(k * K + j) * smax + c) * 2;
    Interval iv; iv.lo = p[0]; iv.hi = p[1];
    return iv;
  }
};

// ---- band mode (Section 2, step (2), read literally) -----------------------------
// The attention map of query scale k, [s_k^2, sum_{i<=k} s_i^2], is cut into parts: the
// first spans the first three key scales (as many of them as the query sees), every later
// key scale is a part of its own.  In a part of n columns query i (flattened, row-major)
// keeps the columns within `radius` of the part's diagonal, floor((2 i + 1) n / (2 s_k^2)).
LV_HD int band_parts(int k) { return k < kMergedScales ? 1 : k - kMergedScales + 2; }
LV_HD int band_part_first(int p) { return p == 0 ? 0 : p + kMergedScales - 1; }
LV_HD int band_part_last(int k, int p) {
  return p == 0 ? (k < kMergedScales - 1 ? k : kMergedScales - 1) : p + kMergedScales - 1;
}

struct BandPart { int tok0, cols, rad; };   // first token, columns, radius (< 0: dense)

template <class Rad>   // Rad(k, j) -> radius of (query scale k, key scale j)
LV_HD BandPart band_part(const Geom& g, const Rad& rad, int k, int p) {
  const int first = band_part_first(p), last = band_part_last(k, p);
  BandPart b;
  b.tok0 = g.off[first]; b.cols = g.off[last + 1] - g.off[first];
  b.rad = last < g.n_sink ? -1 : rad(k, last);
  return b;
}

LV_HD Interval band_interval(const BandPart& b, int nk, int i) {
  Interval iv;
  if (b.rad < 0) { iv.lo = 0; iv.hi = b.cols - 1; return iv; }
  const int ctr = (int)(((uint64_t)(2 * (int64_t)i + 1) * (uint64_t)b.cols) / (uint64_t)(2 * (int64_t)nk));
  iv.lo = ctr - b.rad < 0 ? 0 : ctr - b.rad;
  iv.hi = ctr + b.rad > b.cols - 1 ? b.cols - 1 : ctr + b.rad;
  return iv;
}

struct ArithRad { const HostGeom& g; int operator()(int k, int j) const { return g.rad[k][j]; } };
struct TableRad { const int16_t* rad; int K; LV_HD int operator()(int k, int j) const { return rad[k * K + j]; } };

// ---- groups and patches ------------------------------------------------------------
// Shape (rows x columns of patches, at most nw patches) of the groups that tile a grid of
// pps x pps patches: the fewest groups; among those the most compact shape (a group streams
// the bounding box of its queries' windows), then the taller one.
inline void choose_group_shape(int pps, int nw, int& rh, int& rw) {
  long best = -1;
  rh = 1; rw = 1;
  for (int h = 1; h <= nw && h <= pps; ++h) {
    int w = nw / h; if (w > pps) w = pps;
    const long groups = (long)((pps + h - 1) / h) * ((pps + w - 1) / w);
    const long key = groups * 4096 + (h + w) * 32 + (32 - h);
    if (best < 0 || key < best) { best = key; rh = h; rw = w; }
  }
}

// Shape of a wide patch for scale side s whose groups hold rh x rw patches: at most 32 queries, at most
// eight patches per group, at most twelve rows and columns together (their windows travel in twelve lanes of
// the builder's walk).  The least sum of (rows + 6) (columns + 6) over the scale's patches, which is what
// they keep at a radius of three at equal scale sides; then the wider one, whose keys lie in longer runs.
inline bool choose_wide_shape(int s, int rh, int rw, short& wph, short& wpw) {
  const int H = rh * kPatch < s ? rh * kPatch : s, W = rw * kPatch < s ? rw * kPatch : s;
  long best = -1;
  for (int ph = 1; ph <= H && ph <= 11; ++ph)
    for (int pw = 1; pw <= W && ph * pw <= kWideQueries && ph + pw <= 12; ++pw) {
      if (((H + ph - 1) / ph) * ((W + pw - 1) / pw) > kWidePatches) continue;
      const long ny = s / H * ((H + ph - 1) / ph) + (s % H + ph - 1) / ph;    // whole groups, then the last one
      const long nx = s / W * ((W + pw - 1) / pw) + (s % W + pw - 1) / pw;
      const long key = ny * nx * (ph + 6) * (pw + 6) * 16 - pw;
      if (best < 0 || key < best) { best = key; wph = (short)ph; wpw = (short)pw; }
    }
  return best >= 0;
}

// Order of the rows of a box in the wide patches' key list.  Row by row a box serves its group's patches one
// after the other, and every phase ends when the patch whose rows are passing is done; with the rows dealt from four
// strips in turn, each phase holds keys of all of them.  (Longest wave over the mean, summed over the phases:
// 1.31 -> 1.19 for 256 queries on 680 keys, 1.48 -> 1.31 for side 64 of a 14-scale list.)  The first three chunks
// keep the order of the scales, so that lists that begin with whole scales need no tokens for them.
constexpr int kPlainKeys = 192;
LV_HD bool dealt_box(int mode, int ubase) { return mode == kModeWindow && ubase >= kPlainKeys; }
LV_HD int dealt_row(int i, int rows) {     // row of the box at place i
  const int a = rows >> 2, b = rows & 3, strip = i < 4 * a ? i & 3 : i - 4 * a, round = i < 4 * a ? i >> 2 : a;
  return strip * a + (strip < b ? strip : b) + round;
}

// patches of a group whose steps walk the key list: phase tables, ring offsets and the list's order are theirs
LV_HD int walked_patches(const Geom& g) { return g.n_wide ? g.n_wide : g.NW; }

LV_HD int patches_per_side(const Geom& g, int k) { return (g.s[k] + kPatch - 1) / kPatch; }
LV_HD int scale_patches(const Geom& g, int k) {
  if (g.mode == kModeBand) return (g.s[k] * g.s[k] + kPatchQueries - 1) / kPatchQueries;
  return patches_per_side(g, k) * patches_per_side(g, k);
}
LV_HD int groups_y(const Geom& g, int k) {
  if (g.mode == kModeBand) return (scale_patches(g, k) + g.NW - 1) / g.NW;
  return (patches_per_side(g, k) + g.grh[k] - 1) / g.grh[k];
}
LV_HD int groups_x(const Geom& g, int k) {
  if (g.mode == kModeBand) return 1;
  return (patches_per_side(g, k) + g.grw[k] - 1) / g.grw[k];
}

// group index (inside a head group) -> (query scale, gy, gx)
LV_HD void group_coords(const Geom& g, int grp, int& k, int& gy, int& gx) {
  int i = 0;
  while (i + 1 < g.qe - g.qb && grp >= g.grp_off[i + 1]) ++i;
  k = g.qe - 1 - i;
  const int local = grp - g.grp_off[i];
  const int nx = groups_x(g, k);
  gy = local / nx; gx = local % nx;
}

struct Box { int ylo, yhi, xlo, xhi; };  // inclusive; empty when yhi < ylo

// bounding box in key scale j of the windows of query rows [qy0, qy1] x cols [qx0, qx1]
template <class Win>
LV_HD Box window_box(const Win& win, int k, int j, int qy0, int qy1, int qx0, int qx1) {
  Box b;
  b.ylo = win(k, j, qy0).lo; b.yhi = win(k, j, qy1).hi;
  b.xlo = win(k, j, qx0).lo; b.xhi = win(k, j, qx1).hi;
  return b;
}

// valid queries of a group: rows/cols of the scale's grid (window mode) or the flattened
// query range [qy0, qy1] (band mode; qx0 = qx1 = 0)
struct GroupExtent { int k, qy0, qy1, qx0, qx1; };

LV_HD GroupExtent group_extent(const Geom& g, int k, int gy, int gx) {
  GroupExtent e; e.k = k;
  if (g.mode == kModeBand) {
    const int nk = g.s[k] * g.s[k];
    e.qy0 = gy * g.NW * kPatchQueries;
    e.qy1 = e.qy0 + g.NW * kPatchQueries - 1; if (e.qy1 > nk - 1) e.qy1 = nk - 1;
    e.qx0 = e.qx1 = 0;
    return e;
  }
  e.qy0 = gy * g.grh[k] * kPatch; e.qx0 = gx * g.grw[k] * kPatch;
  e.qy1 = e.qy0 + g.grh[k] * kPatch - 1; if (e.qy1 > g.s[k] - 1) e.qy1 = g.s[k] - 1;
  e.qx1 = e.qx0 + g.grw[k] * kPatch - 1; if (e.qx1 > g.s[k] - 1) e.qx1 = g.s[k] - 1;
  return e;
}

// window mode: (y0, x0) corner and ny x nx valid queries; band mode: y0 = first flattened
// query, nx = number of queries, ny = 1.  ny == 0: no such patch (idle wave)
struct PatchExtent { int y0, x0, ny, nx; };

LV_HD PatchExtent patch_extent(const Geom& g, int k, int gy, int gx, int wave) {
  PatchExtent p;
  const int sk = g.s[k];
  if (g.mode == kModeBand) {
    p.y0 = (gy * g.NW + wave) * kPatchQueries; p.x0 = 0;
    const int left = sk * sk - p.y0;
    if (wave >= g.NW || left <= 0) { p.ny = p.nx = 0; return p; }
    p.ny = 1; p.nx = left < kPatchQueries ? left : kPatchQueries;
    return p;
  }
  const int rh = g.grh[k], rw = g.grw[k];
  const int py = gy * rh + wave / rw, px = gx * rw + wave % rw;
  p.y0 = py * kPatch; p.x0 = px * kPatch;
  if (wave >= rh * rw || p.y0 >= sk || p.x0 >= sk) { p.ny = p.nx = 0; return p; }
  p.ny = sk - p.y0 < kPatch ? sk - p.y0 : kPatch;
  p.nx = sk - p.x0 < kPatch ? sk - p.x0 : kPatch;
  return p;
}

// the same of wide patch `wave` of a group
LV_HD PatchExtent wide_extent(const Geom& g, int k, int gy, int gx, int wave) {
  PatchExtent p;
  const int sk = g.s[k];
  if (g.mode == kModeBand) {
    p.y0 = gy * g.NW * kPatchQueries + wave * kWideQueries; p.x0 = 0;
    const int left = sk * sk - p.y0;
    if (left <= 0) { p.ny = p.nx = 0; return p; }
    p.ny = 1; p.nx = left < kWideQueries ? left : kWideQueries;
    return p;
  }
  const int ph = g.wph[k], pw = g.wpw[k], gh = g.grh[k] * kPatch, gw = g.grw[k] * kPatch;
  const int per_row = ((gw < sk ? gw : sk) + pw - 1) / pw;
  const int y = wave / per_row * ph, x = wave % per_row * pw;      // inside the group
  p.y0 = gy * gh + y; p.x0 = gx * gw + x;
  const int h = sk - gy * gh < gh ? sk - gy * gh : gh, w = sk - gx * gw < gw ? sk - gx * gw : gw;
  if (y >= h || x >= w) { p.ny = p.nx = 0; return p; }
  p.ny = h - y < ph ? h - y : ph;
  p.nx = w - x < pw ? w - x : pw;
  return p;
}

// descriptor fields of a patch: first local query row, row stride of the 4x4 arrangement,
// and the columns that hold a query
LV_HD void patch_queries(const Geom& g, int k, const PatchExtent& p, int& q_base, int& sk, uint32_t& valid) {
  valid = 0;
  if (g.mode == kModeBand) {
    q_base = g.off[k] - g.q0 + p.y0; sk = kPatch;
    valid = p.ny ? (p.nx >= kPatchQueries ? 0xffffu : ((1u << p.nx) - 1u)) : 0u;
    return;
  }
  q_base = g.off[k] - g.q0 + p.y0 * g.s[k] + p.x0; sk = g.s[k];
  for (int n = 0; n < kPatchQueries; ++n)
    if (n / kPatch < p.ny && n % kPatch < p.nx) valid |= 1u << n;
}

// number of keys of a group's union list (band mode)
template <class Rad>
LV_HD int band_union_keys(const Geom& g, const Rad& rad, const GroupExtent& e) {
  const int nk = g.s[e.k] * g.s[e.k];
  int n = 0;
  for (int p = 0; p < band_parts(e.k); ++p) {
    const BandPart b = band_part(g, rad, e.k, p);
    n += band_interval(b, nk, e.qy1).hi - band_interval(b, nk, e.qy0).lo + 1;
  }
  return n;
}

// ---- host sizing: the same steps as the device's walk, counted run by run ---------------
// A step is closed when it holds 32 keys or when the next key's 2^logS-key block lies more
// than A blocks after the block of the step's first key (LDS ring constraint).
// Only the number of keys in each block matters for that, so the counter is fed block by block.
struct StepCounter {
  const int logS, A;
  explicit StepCounter(const Geom& g) : logS(g.logS), A(g.A) {}
  int steps = 0, cnt = 0, first_block = 0;
  // n more keys, all in block blk (a block's keys may come in several parts)
  void block(int blk, int n) {
    if (n <= 0) return;
    if (cnt > 0 && blk - first_block > A) { ++steps; cnt = 0; }
    if (cnt == 0) first_block = blk;
    const int full = (cnt + n - 1) / kStepKeys;          // steps that a further key of the block finds full
    if (full > 0) { first_block = blk; steps += full; cnt -= full * kStepKeys; }
    cnt += n;
  }
  void run(int upos, int n) {              // n consecutive keys of the union list, all kept by some query
    if (n <= 0) return;
    const int end = upos + n, last = (end - 1) >> logS;
    int blk = upos >> logS;
    if (blk == last) { block(blk, n); return; }
    block(blk, ((blk + 1) << logS) - upos);
    // (behind one whole block, a multiple of the step's 32 keys, the next ones leave the count as it is)
    if (++blk < last) {
      block(blk, 1 << logS);
      steps += (last - blk - 1) << (logS - 5); first_block = last - 1;
    }
    block(last, end - (last << logS));
  }
  int finish() { if (cnt > 0) { ++steps; cnt = 0; } return steps; }
};
static_assert(kStepKeys == 32, "whole blocks of 2^logS keys");

// What a patch keeps of one axis of a part: its queries' intervals (both ends grow with the
// query) merged into runs, and their summed length.  One run is [lo, hi]; several stand in a pool, from `first` on.
struct AxisSpan { int lo, hi, kept, n_runs, first; };

// iv(c) for c in [from, to]
template <class Iv>
inline AxisSpan span_of(std::vector<Interval>& pool, int from, int to, Iv iv) {
  Interval run = iv(from);
  AxisSpan a = {run.lo, run.hi, run.hi - run.lo + 1, 1, (int)pool.size()};
  for (int c = from + 1; c <= to; ++c) {
    const Interval x = iv(c);
    a.kept += x.hi - x.lo + 1;
    if (x.lo > run.hi + 1) { pool.push_back(run); run = x; ++a.n_runs; }
    else if (x.hi > run.hi) run.hi = x.hi;
  }
  a.hi = run.hi;
  if (a.n_runs > 1) pool.push_back(run);
  return a;
}

}  // namespace lv
