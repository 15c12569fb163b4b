// Plan construction: host-side validation and sizing, device-side builder kernels
// (tables, places, fill) and the parity exports.
#include "internal.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>
#include <vector>

namespace lv {

// ---- host: descriptor -> geometry ------------------------------------------

static void choose_tiling(Geom& g, int waves, int chunk, int depth, int spare) {
  g.NW = waves;
  g.C = chunk; g.D = depth; g.A = 1;
  // group shape of every scale: 4 x 4 patches (16 x 16 queries) where the scale's patch grid
  // is a multiple of it, otherwise whatever needs the fewest workgroups (a 5 x 5 grid is
  // tiled by two groups of 3 x 5 and 2 x 5 patches rather than by four of 16, 4, 4 and 1)
  for (int k = 0; k < g.K; ++k) {
    int rh, rw;
    choose_group_shape((g.s[k] + kPatch - 1) / kPatch, waves, rh, rw);
    g.grh[k] = (short)rh; g.grw[k] = (short)rw;
    if (waves == 16 && k >= g.qb && k < g.qe) choose_wide_shape(g.s[k], rh, rw, g.wph[k], g.wpw[k]);   // (there is one for every side up to kMaxSide)
  }
  g.NR = g.A + 1 + g.D + spare;
  g.logC = 0;
  while ((1 << g.logC) < g.C) ++g.logC;
  g.logS = g.logC; g.R = g.NR * g.C;
  if (waves == 16) {
    // The 16-patch kernel runs phases of two 64-key chunks (`chunk` = 128 keys) over a ring
    // of five: one chunk of look-back, the two of the phase and the two that are landing.
    // The plan counts in 64-key chunks (phase tables, list padding, ring depth).
    g.C = 64; g.logC = 6; g.logS = 6; g.NR = 5; g.R = 320;
  }
}

litevar_status make_spec(const litevar_mask_desc* d, const litevar_plan_opts* opts, PlanSpec& sp) {
  HostGeom& g = sp.g;
  if (!d) return fail(LITEVAR_E_INVALID_ARG, "desc is NULL");
  if (d->n_scales < 1 || d->n_scales > kMaxScales)
    return fail(LITEVAR_E_INVALID_ARG, "n_scales must be in 1..%d (got %d)", kMaxScales, d->n_scales);
  if (!d->scales) return fail(LITEVAR_E_INVALID_ARG, "scales is NULL");
  memset(&g, 0, sizeof g);
  g.K = d->n_scales;
  int64_t L = 0;
  for (int k = 0; k < g.K; ++k) {
    const int s = d->scales[k];
    if (s < 1 || s > kMaxSide)
      return fail(LITEVAR_E_INVALID_ARG, "scales[%d] = %d outside 1..%d", k, s, kMaxSide);
    g.s[k] = s; g.off[k] = (int)L; L += (int64_t)s * s;
    if (L > (int64_t)1 << 30) return fail(LITEVAR_E_UNSUPPORTED, "sequence longer than 2^30 tokens");
    if (s > g.smax) g.smax = s;
  }
  g.off[g.K] = (int)L; g.L = (int)L;
  if (d->mask_mode != LITEVAR_MASK_WINDOW_2D && d->mask_mode != LITEVAR_MASK_BAND_1D)
    return fail(LITEVAR_E_INVALID_ARG, "unknown mask_mode %d", d->mask_mode);
  g.mode = d->mask_mode == LITEVAR_MASK_BAND_1D ? kModeBand : kModeWindow;

  // radius tables: one per head when radius_per_head is given (heads with equal tables are
  // put into one head group and share its work-list), else one for all heads
  if (d->n_heads < 0 || d->n_heads > kMaxHeads)
    return fail(LITEVAR_E_INVALID_ARG, "n_heads must be in 0..%d (got %d)", kMaxHeads, d->n_heads);
  if ((d->n_heads > 0) != (d->radius_per_head != nullptr))
    return fail(LITEVAR_E_INVALID_ARG, "n_heads and radius_per_head must be given together");
  const int KK = g.K * g.K;
  sp.n_heads = d->n_heads;
  sp.rad_all.clear();
  const int n_tables = d->n_heads > 0 ? d->n_heads : 1;
  int n_hg = 0;
  std::vector<int16_t> tab(KK);
  for (int h = 0; h < n_tables; ++h) {
    for (int k = 0; k < g.K; ++k)
      for (int j = 0; j < g.K; ++j) {
        const int r = d->radius_per_head ? d->radius_per_head[(int64_t)h * KK + k * g.K + j]
                    : d->radius_per_scale_pair ? d->radius_per_scale_pair[k * g.K + j]
                    : d->radius_per_key_scale ? d->radius_per_key_scale[j] : d->radius;
        if (r < LITEVAR_RADIUS_DENSE)
          return fail(LITEVAR_E_INVALID_ARG, "radius %d of key scale %d (query scale %d) is below -1", r, j, k);
        // (entries above the diagonal are never used: normalised so that equal tables compare equal)
        tab[k * g.K + j] = j > k ? (int16_t)0 : (int16_t)(r > kMaxRadius ? kMaxRadius : r);
      }
    int found = -1;
    for (int q = 0; q < n_hg && found < 0; ++q)
      if (memcmp(&sp.rad_all[(size_t)q * KK], tab.data(), KK * sizeof(int16_t)) == 0) found = q;
    if (found < 0) { found = n_hg++; sp.rad_all.insert(sp.rad_all.end(), tab.begin(), tab.end()); }
    sp.head_group[h] = (uint8_t)found;
  }
  g.n_hg = n_hg;
  sp.load_head_group(0);

  if (d->n_sink_scales < 0 || d->n_sink_scales > g.K)
    return fail(LITEVAR_E_INVALID_ARG, "n_sink_scales %d outside 0..%d", d->n_sink_scales, g.K);
  g.n_sink = d->n_sink_scales;
  if (d->q_scale_begin < 0 || d->q_scale_end > g.K || d->q_scale_begin >= d->q_scale_end)
    return fail(LITEVAR_E_INVALID_ARG, "query scale range [%d, %d) is empty or outside [0, %d)",
                d->q_scale_begin, d->q_scale_end, g.K);
  g.qb = d->q_scale_begin; g.qe = d->q_scale_end;
  g.q0 = g.off[g.qb]; g.Lq = g.off[g.qe] - g.q0;

  int waves = opts ? opts->waves_per_group : 0;
  if (waves == 0) {
    int sq = 0;
    for (int k = g.qb; k < g.qe; ++k) if (g.s[k] > sq) sq = g.s[k];
    waves = sq > 8 ? 16 : 4;    // (queries of side <= 8 are one group of 2 x 2 patches: the smaller kernel is quicker)
    // A caller that says how many (batch, head) pairs its launches will have gets smaller
    // groups when 16-patch groups would leave most of the GPU's 256 CUs without a workgroup
    // (measured on the VAR-d30 KV step: 60 pairs 14.4 -> 10.4 us with 4 patches per group, 120
    // pairs 14.8 -> 13.4 us with 8, from 240 pairs on 16 patches per group are the quickest).
    const int hint = opts ? opts->batch_heads_hint : 0;
    if (hint < 0) return fail(LITEVAR_E_INVALID_ARG, "batch_heads_hint must not be negative (got %d)", hint);
    if (waves == 16 && hint > 0) {
      int64_t g16 = 0, g8 = 0;
      for (int k = g.qb; k < g.qe; ++k) {
        const int pps = (g.s[k] + kPatch - 1) / kPatch;
        g16 += (int64_t)((pps + 3) / 4) * ((pps + 3) / 4);
        g8 += (int64_t)((pps + 3) / 4) * ((pps + 1) / 2);
      }
      constexpr int64_t kEnoughWorkgroups = 230;
      if (hint * g16 < kEnoughWorkgroups) waves = hint * g8 >= kEnoughWorkgroups ? 8 : 4;
      // A full sequence of many query scales at a small batch: the launch is as long as its
      // largest workgroup, and a group of 2 x 2 patches streams about half the keys of a
      // group of 4 x 4 (VAR-d16, 32 pairs x 10 scales: 17.7 us with 16 patches per group,
      // 15.0 with 8, 12.4 with 4).
      else if (hint * g16 < 2 * 256 && g.qe - g.qb > 4) waves = 4;
    }
  }
  if (waves != 4 && waves != 8 && waves != 16)
    return fail(LITEVAR_E_INVALID_ARG, "waves_per_group must be 0, 4, 8 or 16 (got %d)", waves);
  int chunk = opts ? opts->chunk_keys : 0, depth = opts ? opts->prefetch_chunks : 0;
  int spare = opts ? opts->spare_chunks : -1;
  if (chunk == 0) chunk = waves == 16 ? 128 : 32;
  if (depth == 0) depth = 2;
  if (spare < 0) spare = waves == 16 ? 0 : chunk == 32 ? 2 : 1;
  if (waves == 16 && (chunk != 128 || depth != 2 || spare != 0))
    return fail(LITEVAR_E_INVALID_ARG, "16 patches per group need (chunk_keys, prefetch_chunks, spare_chunks) = (128, 2, 0)");
  static const int ok[][3] = {{32, 2, 2}, {64, 2, 1}};
  bool found = false;
  for (const auto& t : ok) found |= (t[0] == chunk && t[1] == depth && t[2] == spare);
  found |= waves == 16;
  if (!found)
    return fail(LITEVAR_E_INVALID_ARG, "unsupported (chunk_keys, prefetch_chunks, spare_chunks) = (%d, %d, %d)",
                chunk, depth, spare);
  choose_tiling(g, waves, chunk, depth, spare);
  g.n_wide = waves == 16 && !(opts && opts->patches_per_wave == 1) ? kWidePatches : 0;

  int64_t ng = 0, np = 0;
  for (int i = 0; i < g.qe - g.qb; ++i) {
    const int k = g.qe - 1 - i;
    g.grp_off[i] = (int)ng;
    ng += (int64_t)groups_y(g, k) * groups_x(g, k);
    np += (int64_t)scale_patches(g, k);
  }
  g.grp_off[g.qe - g.qb] = (int)ng;
  if (ng * g.n_hg > (int64_t)1 << 26) return fail(LITEVAR_E_UNSUPPORTED, "too many groups");
  g.n_groups = (int)ng; g.n_patches = (int)np;
  return LITEVAR_OK;
}

static uint64_t align256(uint64_t x) { return (x + 255) & ~(uint64_t)255; }

// The sizing walk visits every block of every group's list on the host (30 tables of 13 x 13 queries: 29 us, 540 key by key).
// Callers size and then build with the same descriptor, often repeatedly,
// so the last result is remembered per thread, keyed by the whole specification.
static thread_local struct { bool valid; PlanSpec sp; PlanSizes z; } g_last_sizing = {false, {}, {}};

static litevar_status size_plan_uncached(PlanSpec& sp, PlanSizes& z);

static bool same_spec(const PlanSpec& a, const PlanSpec& b) {
  // (the Geom holds the radii of the head group that was loaded last: compare it with
  // group 0 loaded on both sides, which is how make_spec leaves it)
  return memcmp(&a.g, &b.g, sizeof a.g) == 0 && a.n_heads == b.n_heads && a.rad_all == b.rad_all &&
         memcmp(a.head_group, b.head_group, sizeof a.head_group) == 0;
}

litevar_status size_plan(PlanSpec& sp, PlanSizes& z) {
  const int asked_wide = sp.g.n_wide;
  if (g_last_sizing.valid && same_spec(g_last_sizing.sp, sp)) {
    z = g_last_sizing.z;
    sp.g.n_wide = z.n_wide;
    sp.group_phases = g_last_sizing.sp.group_phases; sp.patch_counts = g_last_sizing.sp.patch_counts;
    return LITEVAR_OK;
  }
  litevar_status rc = size_plan_uncached(sp, z);
  if (rc == LITEVAR_OK && sp.g.n_wide != asked_wide) rc = size_plan_uncached(sp, z);      // (without wide patches)
  sp.load_head_group(0);
  z.n_wide = sp.g.n_wide;
  if (rc == LITEVAR_OK) {
    g_last_sizing.sp = sp; g_last_sizing.z = z; g_last_sizing.valid = true;
    g_last_sizing.sp.g.n_wide = asked_wide;             // (what the next one is compared with)
  }
  return rc;
}

// a group's box in a key scale: its rows and columns and its first entry in the group's list
struct ListBox { int base, ylo, n_rows, xlo, w; };

// The host's walk over one patch, run by run: bands, and windows with gaps between neighbouring queries
struct PatchWalk {
  StepCounter steps;
  const std::vector<Interval>& pool;
  int64_t pairs = 0;

  // an axis' keys; `from` is the entry of coordinate 0
  void runs(const AxisSpan& a, int from) {
    each_run(a, [&](int lo, int hi) { steps.run(from + lo, hi - lo + 1); });
  }
  template <class F> void each_run(const AxisSpan& a, F f) const {
    if (a.n_runs == 1) f(a.lo, a.hi);
    else for (int i = a.first; i < a.first + a.n_runs; ++i) f(pool[i].lo, pool[i].hi);
  }
  // its keys of one key scale: rows x columns of the group's box, whose rows may be dealt (see dealt_row)
  void box(const AxisSpan& rows, const AxisSpan& cols, const ListBox& b, bool dealt) {
    pairs += (int64_t)rows.kept * cols.kept;
    auto row = [&](int place) { runs(cols, b.base + place * b.w - b.xlo); };
    if (!dealt) { each_run(rows, [&](int lo, int hi) { for (int y = lo; y <= hi; ++y) row(y - b.ylo); }); return; }
    const int per = b.n_rows >> 2, extra = b.n_rows & 3;      // rows of a strip, and how many have one more
    for (int i0 = 0; i0 < b.n_rows; i0 += 64) {
      const int round0 = i0 >> 2;
      uint64_t places = 0;                                    // bit i: place i0 + i holds a row of the patch
      each_run(rows, [&](int lo, int hi) {
        for (int strip = 0; strip < 4; ++strip) {             // place 4 round + strip holds row strip start + round
          const int start = b.ylo + strip * per + std::min(strip, extra), n = per + (strip < extra);
          const int from = std::max(std::max(lo - start, 0), round0), to = std::min(std::min(hi - start, n - 1), round0 + 15);
          if (from > to) continue;
          const uint64_t upto = to - round0 == 15 ? ~0ull : (1ull << (4 * (to - round0) + 4)) - 1;
          places |= (0x1111111111111111ull << strip) & upto & ~((1ull << (4 * (from - round0))) - 1);
        }
      });
      for (; places; places &= places - 1) row(i0 + __builtin_ctzll(places));
    }
  }
};

// The host's walk over all patches of a group whose windows have no gaps, eight patches in the lanes of a vector: how many keys
// of a box's first entries a patch keeps is a product of rows and columns, formed once for every block of the list, and
// the steps follow from the keys in each block as in StepCounter.  (Sizing with a patch at a time, several rows together: 34 240
// tokens 618 us, 30 tables of 16 x 16 queries 76, all pairs of 34 240 tokens 3791; like this 169, 40 and 574.)
// All values are exact modulo 2^16: a block holds at most 64 keys, and a patch keeps some of every box, so that the
// blocks between two of its keys number less than 2^16.
typedef short v8s __attribute__((ext_vector_type(8)));
typedef unsigned short v8u __attribute__((ext_vector_type(8)));
struct GroupWalk {
  static constexpr int kMost = (16 + kWidePatches) / 8;
  const int logS, n_vec, first_wide;                     // vectors in use, and the first that holds wide patches
  const short A;
  v8s n[kMost], cnt[kMost], first[kMost];                // keys of the block at hand, keys and first block of the open step
  v8u closed[kMost];                                     // steps since `steps` was brought up to date
  v8s row_lo[kMost], row_n[kMost], col_lo[kMost], col_w[kMost], before[kMost];
  int steps[8 * kMost]; int64_t pairs[8 * kMost];
  const AxisSpan *rows[8 * kMost], *cols[8 * kMost];     // of key scale 0; scale j's are j strides away
  int row_stride[8 * kMost], col_stride[8 * kMost];
  std::vector<v8s> dealt_rows;                           // by place: the wide patches' rows before it, and whether its row is theirs
  int pending = -1;                                      // block whose keys are in n

  GroupWalk(const Geom& g) : logS(g.logS), n_vec((g.NW + g.n_wide + 7) / 8), first_wide(g.n_wide ? g.NW / 8 : kMost), A((short)g.A) {}
  void start() {
    static const AxisSpan none = {0, -1, 0, 1, 0};
    for (int v = 0; v < kMost; ++v) { n[v] = cnt[v] = first[v] = v8s{}; closed[v] = v8u{}; }
    for (int l = 0; l < 8 * kMost; ++l) { steps[l] = 0; pairs[l] = 0; rows[l] = cols[l] = &none; row_stride[l] = col_stride[l] = 0; }
    pending = -1;
  }
  static v8s sel(v8s mask, v8s a, v8s b) { return (mask & a) | (~mask & b); }
  static v8s clamp(v8s x, v8s hi) { return __builtin_elementwise_min(__builtin_elementwise_max(x, v8s{}), hi); }
  void end_block() {
    const v8s blk = (short)pending;
    for (int v = 0; v < n_vec; ++v) {
      const v8s has = n[v] > (short)0, far = __builtin_bit_cast(v8s, __builtin_bit_cast(v8u, blk - first[v]) > (unsigned short)A);
      const v8s cut = has & (cnt[v] > (short)0) & far;
      cnt[v] &= ~cut;
      const v8s open = cnt[v] + n[v], full = ((open - (short)1) >> (short)5) & has;
      first[v] = sel(has & ((cnt[v] == (short)0) | (full > (short)0)), blk, first[v]);
      cnt[v] = open - (full << (short)5);
      closed[v] += __builtin_bit_cast(v8u, full - cut);
      n[v] = v8s{};
    }
  }
  // the group's box in key scale j
  void box(int j, const ListBox& b, bool dealt) {
    for (int l = 0; l < 8 * n_vec; ++l) {
      const AxisSpan &r = rows[l][j * row_stride[l]], &c = cols[l][j * col_stride[l]];
      row_lo[l >> 3][l & 7] = (short)(r.lo - b.ylo); row_n[l >> 3][l & 7] = (short)(r.hi - r.lo + 1);
      col_lo[l >> 3][l & 7] = (short)(c.lo - b.xlo); col_w[l >> 3][l & 7] = (short)(c.hi - c.lo + 1);
      pairs[l] += (int64_t)r.kept * c.kept;
    }
    if (dealt) {
      const int v = first_wide;
      dealt_rows.resize(2 * (b.n_rows + 1));
      v8s sum = {};
      for (int i = 0; i < b.n_rows; ++i) {
        const v8s at = (v8s)(short)dealt_row(i, b.n_rows) - row_lo[v], its = (at >= (short)0) & (at < row_n[v]);
        dealt_rows[2 * i] = sum; dealt_rows[2 * i + 1] = its;
        sum -= its;
      }
      dealt_rows[2 * b.n_rows] = sum; dealt_rows[2 * b.n_rows + 1] = v8s{};
    }
    for (int v = 0; v < n_vec; ++v) before[v] = v8s{};
    const int end = b.base + b.n_rows * b.w;
    const uint64_t inv = (((uint64_t)1 << 40) + b.w - 1) / b.w;          // i / w = i inv >> 40, exact for i w < 2^40
    static_assert((uint64_t)kMaxSide * kMaxSide * kMaxSide < (uint64_t)1 << 40, "sides");
    for (int blk = b.base >> logS;; ++blk) {
      if (blk != pending) { if (pending >= 0) end_block(); pending = blk; }
      const int stop = std::min((blk + 1) << logS, end), r = (int)((uint64_t)(stop - b.base) * inv >> 40);
      const v8s place = (short)r, x = (short)(stop - b.base - r * b.w);
      for (int v = 0; v < n_vec; ++v) {
        const v8s at = place - row_lo[v];
        v8s whole = clamp(at, row_n[v]), part = (at >= (short)0) & (at < row_n[v]);
        if (dealt && v == first_wide) { whole = dealt_rows[2 * r]; part = dealt_rows[2 * r + 1]; }
        const v8s now = whole * col_w[v] + (part & clamp(x - col_lo[v], col_w[v]));
        n[v] += now - before[v];
        before[v] = now;
      }
      if (stop == end) break;
    }
    for (int v = 0; v < n_vec; ++v) {
      for (int i = 0; i < 8; ++i) steps[8 * v + i] += closed[v][i];
      closed[v] = v8u{};
    }
  }
  void close() {                                         // behind the last box
    if (pending >= 0) end_block();
    for (int v = 0; v < n_vec; ++v)
      for (int i = 0; i < 8; ++i) steps[8 * v + i] += closed[v][i] + (cnt[v][i] > 0);
  }
};

constexpr int kMostPatchSteps = 65535;                  // (counts travel in 16 bits)
constexpr int64_t kMostSteps = (int64_t)1 << 26;

// clears sp.g.n_wide and stops where the wide patches would pass the limits
static litevar_status size_plan_uncached(PlanSpec& sp, PlanSizes& z) {
  HostGeom& g = sp.g;
  sp.group_phases.clear(); sp.patch_counts.clear();
  sp.group_phases.reserve((size_t)g.n_groups * g.n_hg);
  sp.patch_counts.reserve((size_t)g.n_groups * g.n_hg * (g.NW + g.n_wide));
  memset(&z, 0, sizeof z);
  std::vector<Interval> pool;
  std::vector<AxisSpan> ax;            // window mode: [key scale][patch row or column of the query scale]
  std::vector<AxisSpan> wide_rows, wide_cols;   // the same of the wide patches: [key scale][group row, patch row in it]
  std::vector<int64_t> kept_before;    // kept keys of the coordinates (queries of a group) before c, in the part at hand
  std::vector<Interval> of_query;      // band mode: intervals of a group's queries, in the part at hand
  std::vector<PatchWalk> walks;
  GroupWalk together(g);
  // window mode: the windows' centres, which are the same for every head group: [query scale][key scale][coordinate]
  std::vector<int16_t> centres;
  size_t centre_of[kMaxScales] = {};
  for (int k = g.qb; k < g.qe && g.mode == kModeWindow; ++k) {
    centre_of[k] = centres.size();
    for (int j = 0; j <= k; ++j)
      for (int c = 0; c < g.s[k]; ++c) centres.push_back((int16_t)window_interval(g.s[k], g.s[j], c, 0).lo);
  }
  ListBox boxes[kMaxScales];
  for (int hg = 0; hg < g.n_hg; ++hg) {
    sp.load_head_group(hg);
    const ArithRad rad{g};
    int64_t pairs_hg = 0;
    for (int k = g.qe - 1; k >= g.qb; --k) {
      const int pps = patches_per_side(g, k), nk = g.s[k] * g.s[k];
      const int ngy = groups_y(g, k), ngx = groups_x(g, k);
      const bool wide = g.n_wide > 0;
      // wide patch rows of a group, and columns (window mode)
      int wny = 0, wnx = 0;
      bool gaps = true;
      if (g.mode == kModeWindow) {
        const int gh = g.grh[k] * kPatch, gw = g.grw[k] * kPatch, ph = g.wph[k], pw = g.wpw[k], sk = g.s[k];
        ax.resize((size_t)(k + 1) * pps);
        if (wide) {
          wny = ((gh < sk ? gh : sk) + ph - 1) / ph; wnx = ((gw < sk ? gw : sk) + pw - 1) / pw;
          wide_rows.resize((size_t)(k + 1) * ngy * wny);
          wide_cols.resize((size_t)(k + 1) * ngx * wnx);
        }
        pool.clear();
        gaps = false;
        kept_before.resize(sk + 1);
        const int16_t* ctr = &centres[centre_of[k]];
        for (int j = 0; j <= k; ++j, ctr += sk) {
          const int sj = g.s[j], last = sj - 1, r = j < g.n_sink ? -1 : g.rad[k][j];
          auto window = [&](int c) {
            if (r < 0) return Interval{0, last};
            return Interval{ctr[c] - r < 0 ? 0 : ctr[c] - r, ctr[c] + r > last ? last : ctr[c] + r};
          };
          // (neighbouring centres are ceil(sj / sk) apart at most: windows as wide as that leave no gaps)
          const bool joined = r < 0 || sj <= (int64_t)(2 * r + 1) * sk;
          gaps = gaps || !joined;
          if (joined) {
            int64_t n = 0;
            for (int c = 0; c < sk; ++c) { kept_before[c] = n; const Interval iv = window(c); n += iv.hi - iv.lo + 1; }
            kept_before[sk] = n;
          }
          auto span = [&](int from, int to) {
            if (joined) return AxisSpan{window(from).lo, window(to).hi, (int)(kept_before[to + 1] - kept_before[from]), 1, 0};
            return span_of(pool, from, to, window);
          };
          // patches of `side` coordinates, in groups of `group`
          auto cut = [&](AxisSpan* a, int group, int per_group, int side) {
            for (int y = 0; y < sk; y += group, a += per_group)
              for (int p = 0, c = y, end = std::min(sk, y + group); c < end; ++p, c += side) a[p] = span(c, std::min(end, c + side) - 1);
          };
          cut(&ax[(size_t)j * pps], sk, pps, kPatch);
          if (!wide) continue;
          cut(&wide_rows[(size_t)j * ngy * wny], gh, wny, ph);
          cut(&wide_cols[(size_t)j * ngx * wnx], gw, wnx, pw);
        }
      }
      for (int gi = 0; gi < ngy * ngx; ++gi) {
        const int gy = gi / ngx, gx = gi % ngx;
        const GroupExtent e = group_extent(g, k, gy, gx);
        int nu = 0;
        if (g.mode == kModeBand) {
          nu = band_union_keys(g, rad, e);
        } else {
          for (int j = 0; j <= k; ++j) {
            const AxisSpan* a = &ax[(size_t)j * pps];
            ListBox& b = boxes[j];
            b.base = nu;
            b.ylo = a[e.qy0 / kPatch].lo; b.n_rows = a[e.qy1 / kPatch].hi - b.ylo + 1;
            b.xlo = a[e.qx0 / kPatch].lo; b.w = a[e.qx1 / kPatch].hi - b.xlo + 1;
            nu += b.n_rows * b.w;
          }
        }
        const int nph = (nu + g.C - 1) / g.C;
        z.n_union += (int64_t)nph * g.C;
        z.n_phase_entries += (int64_t)nph * walked_patches(g);
        sp.group_phases.push_back(nph);
        const int n_walks = g.NW + g.n_wide;
        auto extent = [&](int w) { return w < g.NW ? patch_extent(g, k, gy, gx, w) : wide_extent(g, k, gy, gx, w - g.NW); };
        if (gaps) {
          walks.clear();
          for (int w = 0; w < n_walks; ++w) walks.push_back(PatchWalk{StepCounter(g), pool});
        }
        if (g.mode == kModeBand) {
          int ubase = 0;
          for (int pt = 0; pt < band_parts(k); ++pt) {
            const BandPart b = band_part(g, rad, k, pt);
            const int n = e.qy1 - e.qy0 + 1;
            of_query.resize(n); kept_before.resize(n + 1);
            kept_before[0] = 0;
            // band_interval of every query; the centre moves by 2 cols / 2 nk, the remainder kept
            const int64_t den = 2 * (int64_t)nk, num = (2 * (int64_t)e.qy0 + 1) * b.cols, by = 2 * (int64_t)b.cols;
            int64_t ctr = num / den, rem = num % den;
            const int64_t ctr_by = by / den, rem_by = by % den;
            for (int i = 0; i < n; ++i) {
              Interval& iv = of_query[i];
              if (b.rad < 0) iv = {0, b.cols - 1};
              else iv = {(int)std::max<int64_t>(ctr - b.rad, 0), (int)std::min<int64_t>(ctr + b.rad, b.cols - 1)};
              kept_before[i + 1] = kept_before[i] + iv.hi - iv.lo + 1;
              ctr += ctr_by; rem += rem_by;
              if (rem >= den) { rem -= den; ++ctr; }
            }
            const int glo = of_query.front().lo, ghi = of_query.back().hi;
            pool.clear();
            const bool joined = b.rad < 0 || b.cols <= (2 * (int64_t)b.rad + 1) * nk;       // (as in window mode)
            for (int w = 0; w < n_walks; ++w) {
              const PatchExtent p = extent(w);
              if (p.ny == 0) continue;
              const int from = p.y0 - e.qy0, to = from + p.nx - 1;
              walks[w].runs(joined ? AxisSpan{of_query[from].lo, of_query[to].hi, 0, 1, 0}
                                   : span_of(pool, from, to, [&](int i) { return of_query[i]; }), ubase - glo);
              walks[w].pairs += kept_before[to + 1] - kept_before[from];
            }
            ubase += ghi - glo + 1;
          }
        } else {
          if (!gaps) together.start();
          for (int w = 0; w < n_walks; ++w) {
            const PatchExtent p = extent(w);
            if (p.ny == 0) continue;
            const int v = w - g.NW, row_stride = v < 0 ? pps : ngy * wny, col_stride = v < 0 ? pps : ngx * wnx;
            const AxisSpan* rows = v < 0 ? &ax[p.y0 / kPatch] : &wide_rows[gy * wny + v / wnx];
            const AxisSpan* cols = v < 0 ? &ax[p.x0 / kPatch] : &wide_cols[gx * wnx + v % wnx];
            if (!gaps) {
              together.rows[w] = rows; together.row_stride[w] = row_stride;
              together.cols[w] = cols; together.col_stride[w] = col_stride;
              continue;
            }
            for (int j = 0; j <= k; ++j, rows += row_stride, cols += col_stride)
              walks[w].box(*rows, *cols, boxes[j], v >= 0 && dealt_box(g.mode, boxes[j].base));
          }
          if (!gaps) {
            for (int j = 0; j <= k; ++j) together.box(j, boxes[j], wide && dealt_box(g.mode, boxes[j].base));
            together.close();
          }
        }
        for (int w = 0; w < n_walks; ++w) {
          const int ns = gaps ? walks[w].steps.finish() : together.steps[w];
          const int64_t pairs = gaps ? walks[w].pairs : together.pairs[w];
          if (w < g.NW) {
            if (ns > kMostPatchSteps) return fail(LITEVAR_E_UNSUPPORTED, "a query patch needs more than 65535 steps");
            z.n_steps += ns; pairs_hg += pairs;
          } else {
            z.n_wide_steps += ns;
            if (ns > kMostPatchSteps || z.n_wide_steps > kMostSteps) { g.n_wide = 0; return LITEVAR_OK; }
          }
          sp.patch_counts.push_back({(uint16_t)ns, (uint8_t)(pairs % kPairsModulus)});
        }
      }
    }
    z.retained_pairs += pairs_hg;
    if (hg < kMaxHeads) z.pairs_of_group[hg] = pairs_hg;
  }
  if (z.n_steps > kMostSteps || z.n_union > (int64_t)1 << 30)
    return fail(LITEVAR_E_UNSUPPORTED, "work-list too large (%lld steps)", (long long)z.n_steps);
  const uint64_t ngt = (uint64_t)g.n_groups * g.n_hg;
  uint64_t o = 0;
  z.off[kSecHeader] = o; o += sizeof(Header);
  z.off[kSecWin] = o;
  o = align256(o + (g.mode == kModeWindow ? (uint64_t)g.n_hg * g.K * g.K * g.smax * 2 * sizeof(int16_t) : 0));
  z.off[kSecRad] = o; o = align256(o + (uint64_t)g.n_hg * g.K * g.K * sizeof(int16_t));
  z.off[kSecHeadMap] = o; o = align256(o + (uint64_t)kMaxHeads * sizeof(int32_t));
  z.off[kSecGroups] = o; o = align256(o + ngt * sizeof(GroupDesc));
  z.off[kSecWaves] = o; o = align256(o + ngt * (g.NW + g.n_wide) * sizeof(WaveDesc));
  z.off[kSecPhaseEnd] = o; o = align256(o + (uint64_t)z.n_phase_entries * sizeof(int32_t));
  z.off[kSecUnion] = o; o = align256(o + (uint64_t)z.n_union * sizeof(int32_t));
  z.off[kSecStepAddr] = o; o = align256(o + (uint64_t)(g.n_wide ? z.n_wide_steps * kWideDesc : z.n_steps * (int64_t)sizeof(uint2)) * 64);
  z.off[kSecStepMask] = o; o = align256(o + (uint64_t)z.n_steps * 8 * sizeof(uint64_t));
  z.off[kSecStepTok] = o; o = align256(o + (uint64_t)z.n_steps * kStepKeys * sizeof(int32_t));
  z.off[kSecEnd] = o;
  z.bytes = o;
  return LITEVAR_OK;
}

// ---- device: builder kernels -------------------------------------------------

struct BlobPtrs {
  Header* hdr; int16_t* win; int16_t* rad; int32_t* head_map; GroupDesc* groups; WaveDesc* waves;
  int32_t* phase_end; int32_t* union_tok; uint2* step_addr; uint64_t* step_mask; int32_t* step_tok;
};

static BlobPtrs blob_ptrs(void* blob, const uint64_t* off) {
  char* b = (char*)blob;
  BlobPtrs p;
  p.hdr = (Header*)(b + off[kSecHeader]); p.win = (int16_t*)(b + off[kSecWin]);
  p.rad = (int16_t*)(b + off[kSecRad]); p.head_map = (int32_t*)(b + off[kSecHeadMap]);
  p.groups = (GroupDesc*)(b + off[kSecGroups]); p.waves = (WaveDesc*)(b + off[kSecWaves]);
  p.phase_end = (int32_t*)(b + off[kSecPhaseEnd]); p.union_tok = (int32_t*)(b + off[kSecUnion]);
  p.step_addr = (uint2*)(b + off[kSecStepAddr]); p.step_mask = (uint64_t*)(b + off[kSecStepMask]);
  p.step_tok = (int32_t*)(b + off[kSecStepTok]);
  return p;
}

struct Caps { int64_t n_steps, n_union, n_phase_entries, retained_pairs, n_wide_steps; uint64_t bytes; int n_groups; };

// Where the patches and groups of a plan go.  The host counts the steps of every patch anyway, so the counts travel with
// the builder's launches and nothing is counted on the device: with k_fill's own arguments where all of them
// fit, else ahead of it with k_place's, as many groups to a launch as the 4 KiB argument block takes: 66 of 16 patches.
// All launches of a build, with counting walks and a scan on the device / like this (and before there were wide patches):
// 34 240 tokens 174 / 82 us (103), 36 tables of 2240 tokens 252 / 143 (154).  A launch of k_place takes 3.3.
// A list's words: first step, first wide step and first phase of every group, the phases up to its end, and for every patch
// a Count of its steps and its kept pairs modulo 251 (the wide patches after the others): 16 bits where no patch has
// more than 255 steps, else 32.  A walk that ends at other steps or pairs than the host's marks the plan (a wrong mask
// bit is a wrong pair; a difference of a multiple of 251 in every patch that it touches passes).
struct SmallCount {
  uint16_t v;
  static constexpr int kMost = 255;
  __host__ __device__ static SmallCount of(int steps, int pairs) { return {(uint16_t)(steps | pairs << 8)}; }
  __host__ __device__ int steps() const { return v & 0xff; }
  __host__ __device__ int pairs() const { return v >> 8; }
};
struct LargeCount {
  uint32_t v;
  __host__ __device__ static LargeCount of(int steps, int pairs) { return {(uint32_t)steps | (uint32_t)pairs << 16}; }
  __host__ __device__ int steps() const { return (int)(v & 0xffff); }
  __host__ __device__ int pairs() const { return (int)(v >> 16); }
};
template <int N> struct PlaceList {
  int first_group, n_groups;
  uint32_t w[N];
  template <class Count> __host__ __device__ const Count* counts() const { return (const Count*)(w + 3 * n_groups + 1); }
  __host__ __device__ int phases_of(int i) const { return (int)(w[i + 1 < n_groups ? 3 * i + 5 : 3 * n_groups] - w[3 * i + 2]); }
};
constexpr int kInlineWords = (4096 - sizeof(Geom) - sizeof(BlobPtrs) - sizeof(Caps) - 40) / 4;
constexpr int kLaunchWords = (4096 - sizeof(BlobPtrs) - 40) / 4;
using Places = PlaceList<kInlineWords>;
struct NoPlaces {};
static_assert(sizeof(Places) + sizeof(Geom) + sizeof(BlobPtrs) + sizeof(Caps) + 16 <= 4096, "kernel argument block");
static_assert(sizeof(PlaceList<kLaunchWords>) + sizeof(BlobPtrs) + 24 <= 4096, "kernel argument block");

// groups that fit into `words` words, with `per` patches each
template <class Count> static int groups_in(int words, int per) { return (int)((4 * words - 8) / (12 + per * sizeof(Count))); }

// Where the next group's steps, wide steps and phases begin
struct PlaceAt { uint32_t step[2] = {0, 0}, phase = 0; };

// the groups from `first` on, as many as there are and fit; `at` moves behind them
template <class Count, int N> static void fill_list(const PlanSpec& sp, int first, PlaceAt& at, PlaceList<N>& list) {
  const int per = sp.g.NW + sp.g.n_wide, n_all = (int)sp.group_phases.size();
  list.first_group = first;
  list.n_groups = std::min(n_all - first, groups_in<Count>(N, per));
  uint32_t* w = list.w;
  Count* c = (Count*)(w + 3 * list.n_groups + 1);
  const PlanSpec::PatchCount* count = sp.patch_counts.data() + (size_t)first * per;
  for (int i = 0; i < list.n_groups; ++i) {
    *w++ = at.step[0]; *w++ = at.step[1]; *w++ = at.phase;
    at.phase += (uint32_t)sp.group_phases[first + i];
    for (int j = 0; j < per; ++j, ++count) {
      at.step[j >= sp.g.NW] += count->steps;
      *c++ = Count::of(count->steps, count->pairs);
    }
  }
  *w = at.phase;
}

__device__ inline int sum_of_lanes(int v) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d);
  return v;
}

// K1: the radius tables rad[hg][k][j] (-1: dense part), in window mode the window tables
// win[hg][k][j][c] = inclusive [lo, hi] ((-1,-1) where undefined), and the head map.  Every other
// builder kernel reads these tables and never the radii of the descriptor.
// The radii travel as kernel arguments (no copy that a caller's stream would have to order), the
// lower triangles of as many head groups as fit the 4 KiB argument block: 33 of ten scales, 3 of
// thirty-two.  Thirty distinct tables of ten scales take 3.9 us in one launch; a launch per table
// took 30 x 3.1 us on the GPU.
constexpr int kTableRadii = 1840;
struct TablesArg {
  int K, mode, n_sink, smax, hg0, n_hg, n_heads;   // head groups [hg0, hg0 + n_hg); n_heads < 0: no head map in this launch
  uint16_t s[kMaxScales];
  uint8_t head_group[kMaxHeads];
  int16_t rad[kTableRadii];                        // [hg - hg0][k (k + 1) / 2 + j]
};
static_assert(sizeof(TablesArg) + 4 * sizeof(void*) <= 4096, "kernel argument block");

// grid (entries of a head group's window table / 256, head groups of the launch)
__global__ __launch_bounds__(256) void k_tables(TablesArg a, int16_t* win, int16_t* rad, int32_t* head_map, Header* hdr) {
  const int idx = blockIdx.x * 256 + threadIdx.x, hg = a.hg0 + blockIdx.y;
  if (blockIdx.x == 0 && blockIdx.y == 0 && a.n_heads >= 0) {
    head_map[threadIdx.x] = (int)threadIdx.x < a.n_heads ? a.head_group[threadIdx.x] : 0;
    if (threadIdx.x == 0) hdr->error = kErrNone;       // (k_fill without a count ahead of it marks what it finds wrong)
  }
  const int16_t* r = a.rad + blockIdx.y * (a.K * (a.K + 1) / 2);
  if (idx < a.K * a.K) {
    const int k = idx / a.K, j = idx - k * a.K;
    rad[(size_t)hg * a.K * a.K + idx] = j > k ? (int16_t)0 : j < a.n_sink ? (int16_t)-1 : r[k * (k + 1) / 2 + j];
  }
  if (a.mode != kModeWindow) return;
  const int total = a.K * a.K * a.smax;
  if (idx >= total) return;
  const int c = idx % a.smax, kj = idx / a.smax, k = kj / a.K, j = kj - k * a.K;
  Interval iv = {-1, -1};
  if (j <= k && c < a.s[k]) iv = window_interval(a.s[k], a.s[j], c, j < a.n_sink ? -1 : r[k * (k + 1) / 2 + j]);
  int16_t* out = win + ((size_t)hg * total + idx) * 2;
  out[0] = (int16_t)iv.lo; out[1] = (int16_t)iv.hi;
}
static_assert(kMaxHeads == 256, "one thread per head");

// value of `v` in lane `lane`, for a lane index that is the same in every lane of the wave:
// v_readlane_b32, where __shfl would go through the LDS crossbar
__device__ inline int lane_value(int v, int lane) {
  return __builtin_amdgcn_readlane(v, __builtin_amdgcn_readfirstlane(lane));
}

// Placement of the kept keys of one pass (64 candidate keys, one per lane, in key order) in
// the patch's steps: they get consecutive places; a pass is cut where a step fills up (32
// keys) or where the next key's 2^logS-key block lies more than A blocks after the block of
// the step's first key, exactly as in the host's StepCounter, so both produce the same steps.
// Sink receives
//   keys(step, idx, upos, token, qmask, take)   per pass segment: lanes with take set hold
//                                               the key that becomes entry idx of the step
//   close(step, n_keys, last_upos)              when a step is complete (wave-uniform)
template <class Sink>
struct WavePacker {
  const Geom& g; Sink& sink; int lane;
  int step = 0, cnt = 0, first_block = 0, last_upos = 0;
  __device__ void pass(bool kept, int upos, int tok, unsigned qmask) {
    const uint64_t lt_mask = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    const int blk = upos >> g.logS;
    uint64_t km = __ballot(kept);                     // kept keys of this pass not yet placed
    while (km) {
      const int fl = __builtin_ctzll(km);
      const int fblk = lane_value(blk, fl);
      if (cnt > 0 && fblk - first_block > g.A) { sink.close(step, cnt, last_upos); ++step; cnt = 0; }
      if (cnt == 0) first_block = fblk;
      const bool mine = (km >> lane) & 1;
      // lanes whose key still fits the step's span (blocks grow with the lane), ranked
      const uint64_t fit = __ballot(mine && blk - first_block <= g.A);
      const int rank = __builtin_popcountll(fit & lt_mask);
      const bool take = ((fit >> lane) & 1) && rank < kStepKeys - cnt;
      const uint64_t tm = __ballot(take);
      sink.keys(step, cnt + rank, upos, tok, qmask, take);
      last_upos = lane_value(upos, 63 - __builtin_clzll(tm));
      cnt += __builtin_popcountll(tm);
      km &= ~tm;
      if (cnt == kStepKeys) { sink.close(step, cnt, last_upos); ++step; cnt = 0; }
    }
  }
  __device__ int finish() {
    if (cnt > 0) { sink.close(step, cnt, last_upos); ++step; cnt = 0; }
    return step;
  }
};

// One key scale of the walk over a wide patch (window mode): ny + nx <= 12 lanes from l0 on hold the windows of its
// query rows and columns, the last four of the sixteen those of the group's first and last row and column.
// The rows of the box that some query keeps are closed up in lanes, each with the queries that keep it; a lane's column
// is the same in every pass, so its queries are found once.
template <class Sink>
__device__ int wave_walk_wide_box(const PatchExtent& p, const Interval& mine, int l0, int sj, int offj, int ubase,
                                  WavePacker<Sink>& pack, int lane) {
  const int gylo = lane_value(mine.lo, l0 + 12), gyhi = lane_value(mine.hi, l0 + 13);
  const int gxlo = lane_value(mine.lo, l0 + 14), gw = lane_value(mine.hi, l0 + 15) - gxlo + 1;
  const int ylo = lane_value(mine.lo, l0), yhi = lane_value(mine.hi, l0 + p.ny - 1);
  const int xlo = lane_value(mine.lo, l0 + p.ny), xhi = lane_value(mine.hi, l0 + p.ny + p.nx - 1);
  const int W = xhi - xlo + 1, WL = W < 64 ? W : 64, RP = 64 / WL;
  const int ry = lane / WL, xx = lane - ry * WL;
  auto keeping = [&](int c, int from, int n) {          // the queries of lanes [from, from + n) whose windows hold c
    unsigned bits = 0;
    for (int d = 0; d < n; ++d) bits |= (unsigned)(c >= lane_value(mine.lo, from + d) && c <= lane_value(mine.hi, from + d)) << d;
    return bits;
  };
  unsigned cb = keeping(xlo + xx, l0 + p.ny, p.nx);
  // places of the box's rows in the list: the patch's own rows, or all of them where they are dealt
  const bool dealt = dealt_box(kModeWindow, ubase);
  const int n_rows = gyhi - gylo + 1, i_lo = dealt ? 0 : ylo - gylo, i_hi = dealt ? n_rows - 1 : yhi - gylo;
  for (int i0 = i_lo; i0 <= i_hi; i0 += 64) {
    const int at = min(i0 + lane, i_hi), y_at = gylo + (dealt ? dealt_row(at, n_rows) : at);
    const unsigned rb_at = i0 + lane <= i_hi ? keeping(y_at, l0, p.ny) : 0;
    const uint64_t kept = __ballot(rb_at != 0);
    const int n_kept = __builtin_popcountll(kept), rank = __builtin_popcountll(kept & ((1ull << lane) - 1));
    static_assert(kMaxSide <= 1024, "a row's place and coordinate in ten bits each");
    // (lanes without a kept row all write to lane 63, which then is beyond the kept ones)
    const unsigned rows = (unsigned)__builtin_amdgcn_ds_permute(4 * (rb_at ? rank : 63), (int)(at | y_at << 10 | rb_at << 20));
    for (int r0 = 0; r0 < n_kept; r0 += RP) {
      const unsigned row = (unsigned)__shfl((int)rows, (r0 + ry) & 63);
      const bool in_box = ry < RP && r0 + ry < n_kept;
      const unsigned rb = row >> 20;
      const int urow = ubase + (int)(row & 1023) * gw - gxlo, trow = offj + (int)((row >> 10) & 1023) * sj;
      for (int x0 = xlo; x0 <= xhi; x0 += WL) {
        const int x = x0 + xx;
        if (W > 64) cb = keeping(x, l0 + p.ny, p.nx);
        pack.pass(in_box && x <= xhi && cb, urow + x, trow + x, rb | (cb << p.ny));
      }
    }
  }
  return n_rows * gw;
}

// The walk over a patch's kept keys in the order of its group's list: the 64 lanes of a wave take 64
// consecutive candidate keys at a time (window mode: several rows of a narrow box, or 64 columns of one row of the
// patch's box in a key scale; band mode: 64 columns of the patch's range in a part).
// WIDE: a wide patch.
template <bool WIDE, class Sink>
__device__ int wave_walk_patch(const Geom& g, const TableWin& win, const TableRad& rad, const GroupExtent& e,
                               const PatchExtent& p, Sink& sink, int lane) {
  constexpr int kQ = WIDE ? kWideQueries : kPatchQueries;
  if (p.ny == 0) return 0;
  WavePacker<Sink> pack{g, sink, lane};
  int ubase = 0;
  if (g.mode == kModeBand) {
    const int nk = g.s[e.k] * g.s[e.k];
    for (int pt = 0; pt < band_parts(e.k); ++pt) {
      const BandPart b = band_part(g, rad, e.k, pt);
      const int glo = band_interval(b, nk, e.qy0).lo, ghi = band_interval(b, nk, e.qy1).hi;
      // the queries' intervals: one lane each (a 64-bit division).  Neither end ever falls from one query to the next,
      // so the queries that keep a column are those from the first whose end reaches it to the last that has begun.
      constexpr int kNone = 0x7fffffff;
      Interval mine = {kNone, kNone};
      if (lane < p.nx) mine = band_interval(b, nk, p.y0 + lane);
      const int clo = lane_value(mine.lo, 0), chi = lane_value(mine.hi, p.nx - 1);
      auto up_to = [&](int v, int c) {                  // lanes of the first kQ, in ascending order, with a value of at most c
        int n = 0;
#pragma unroll
        for (int d = kQ / 2; d > 0; d >>= 1) n += __shfl(v, n + d - 1) <= c ? d : 0;
        return n + (int)(__shfl(v, n) <= c);
      };
      for (int c0 = clo; c0 <= chi; c0 += 64) {
        const int c = c0 + lane;
        const unsigned begun = (unsigned)((1ull << up_to(mine.lo, c)) - 1), ended = (unsigned)((1ull << up_to(mine.hi, c - 1)) - 1);
        const unsigned qmask = c <= chi ? begun & ~ended : 0;
        pack.pass(qmask != 0, ubase + c - glo, b.tok0 + c, qmask);
      }
      ubase += ghi - glo + 1;
    }
    return pack.finish();
  }
  // The twelve window intervals that a key scale needs (four patch rows, four patch columns,
  // the group's first and last row and column) are fetched from the table for ALL key scales
  // before the walk: sixteen lanes per key scale, four key scales per round, so the walk pays
  // the table's latency once and not once per key scale.  They are handed round with
  // v_readlane.
  constexpr int kRounds = kMaxScales / 4;
  Interval pre[kRounds];
  // (likewise the key scales' sides and offsets, one per lane)
  const int my_side = g.s[min(lane, g.K - 1)], my_off = g.off[min(lane, g.K - 1)];
  {
    const int sk = g.s[e.k];
    const int role = lane & 15;
    int cq = WIDE ? (role < p.ny ? p.y0 + role : role < p.ny + p.nx ? p.x0 + role - p.ny
                     : role < 12 ? p.y0 : role == 12 ? e.qy0 : role == 13 ? e.qy1 : role == 14 ? e.qx0 : e.qx1)
             : role < 4 ? p.y0 + role : role < 8 ? p.x0 + role - 4 : role == 8 ? e.qy0 : role == 9 ? e.qy1 : role == 10 ? e.qx0 : e.qx1;
    cq = cq < sk ? cq : sk - 1;
#pragma unroll
    for (int t = 0; t < kRounds; ++t) {
      pre[t].lo = 1; pre[t].hi = 0;
      const int j = 4 * t + (lane >> 4);
      if (4 * t <= e.k && j <= e.k && role < (WIDE ? 16 : 12)) pre[t] = win(e.k, j, cq);
    }
  }
  for (int j = 0; j <= e.k; ++j) {
    Interval mine_iv = pre[0];
#pragma unroll
    for (int t = 1; t < kRounds; ++t)
      if ((j >> 2) == t) mine_iv = pre[t];             // (uniform)
    const int l0 = (j & 3) * 16;                         // first lane of this key scale's sixteen
    if constexpr (WIDE) {
      ubase += wave_walk_wide_box(p, mine_iv, l0, lane_value(my_side, j), lane_value(my_off, j), ubase, pack, lane);
      continue;
    }
    const Interval none = {1, 0};
    Interval rw[kPatch], cw[kPatch];
#pragma unroll
    for (int d = 0; d < kPatch; ++d) {
      const Interval r = {lane_value(mine_iv.lo, l0 + d), lane_value(mine_iv.hi, l0 + d)};
      const Interval cc = {lane_value(mine_iv.lo, l0 + 4 + d), lane_value(mine_iv.hi, l0 + 4 + d)};
      rw[d] = d < p.ny ? r : none;
      cw[d] = d < p.nx ? cc : none;
    }
    Box gb, pb;
    gb.ylo = lane_value(mine_iv.lo, l0 + 8); gb.yhi = lane_value(mine_iv.hi, l0 + 9);
    gb.xlo = lane_value(mine_iv.lo, l0 + 10); gb.xhi = lane_value(mine_iv.hi, l0 + 11);
    pb.ylo = rw[0].lo; pb.yhi = lane_value(mine_iv.hi, l0 + p.ny - 1);
    pb.xlo = cw[0].lo; pb.xhi = lane_value(mine_iv.hi, l0 + 4 + p.nx - 1);
    const int gw = gb.xhi - gb.xlo + 1;
    const int sj = lane_value(my_side, j), offj = lane_value(my_off, j);
    // lanes of a pass in key order: RP rows of the patch's box (W columns each) when the box
    // is narrower than a wave, else 64 columns of one row
    const int W = pb.xhi - pb.xlo + 1;
    const int WL = W < 64 ? W : 64, RP = 64 / WL;
    const int ry = lane / WL, xx = lane - ry * WL;
    for (int y0 = pb.ylo; y0 <= pb.yhi; y0 += RP) {
      const int y = y0 + ry;
      unsigned rb = 0;
      if (ry < RP && y <= pb.yhi) {
#pragma unroll
        for (int d = 0; d < kPatch; ++d) rb |= (unsigned)(y >= rw[d].lo && y <= rw[d].hi) << d;
      }
      const unsigned rowmask = ((rb & 1) ? 0x000fu : 0u) | ((rb & 2) ? 0x00f0u : 0u) |
                               ((rb & 4) ? 0x0f00u : 0u) | ((rb & 8) ? 0xf000u : 0u);
      const int urow = ubase + (y - gb.ylo) * gw - gb.xlo, trow = offj + y * sj;
      for (int x0 = pb.xlo; x0 <= pb.xhi; x0 += WL) {
        const int x = x0 + xx;
        unsigned cb = 0;
        if (rb && x <= pb.xhi) {
#pragma unroll
          for (int d = 0; d < kPatch; ++d) cb |= (unsigned)(x >= cw[d].lo && x <= cw[d].hi) << d;
        }
        pack.pass(cb != 0, urow + x, trow + x, (cb * 0x1111u) & rowmask);
      }
    }
    ubase += (gb.yhi - gb.ylo + 1) * gw;
  }
  return pack.finish();
}

// the tables of the head group that global group G belongs to
struct GroupTables { TableWin win; TableRad rad; int grp; };
__device__ inline GroupTables group_tables(const Geom& g, const BlobPtrs& p, int G) {
  const int hg = G / g.n_groups;
  GroupTables t;
  t.win = TableWin{p.win + (size_t)hg * g.K * g.K * g.smax * 2, g.K, g.smax};
  t.rad = TableRad{p.rad + (size_t)hg * g.K * g.K, g.K};
  t.grp = G - hg * g.n_groups;
  return t;
}

// a patch's descriptor without what its walk and its place in the plan say
__device__ inline WaveDesc patch_desc(const Geom& g, int k, const PatchExtent& pe) {
  WaveDesc wd;
  int q_base, sk; uint32_t valid;
  patch_queries(g, k, pe, q_base, sk, valid);
  wd.step_begin = 0; wd.n_steps = 0;
  wd.q_base = q_base;
  wd.sk = (int16_t)sk; wd.ny = (int16_t)pe.ny; wd.nx = (int16_t)pe.nx; wd.kq = (int16_t)k;
  wd.pairs = 0; wd.valid = valid; wd.first_ends = 0;
  return wd;
}
__device__ inline WaveDesc wide_desc(const Geom& g, int k, const PatchExtent& pe) {
  WaveDesc wd;
  const int n = pe.ny * pe.nx;
  wd.step_begin = 0; wd.n_steps = 0;
  wd.q_base = g.off[k] - g.q0 + (g.mode == kModeBand ? pe.y0 : pe.y0 * g.s[k] + pe.x0);
  wd.sk = (int16_t)(g.mode == kModeBand ? 0 : g.s[k]); wd.ny = (int16_t)pe.ny; wd.nx = (int16_t)pe.nx; wd.kq = (int16_t)k;
  wd.pairs = pe.nx ? (65536 + pe.nx - 1) / pe.nx : 0;
  wd.valid = n >= 32 ? 0xffffffffu : (1u << n) - 1u; wd.first_ends = 0;
  return wd;
}

// a group's descriptor without its place in the plan, by one wave
__device__ GroupDesc group_desc(const Geom& g, const GroupTables& t, int k, int gy, int gx, int lane) {
  const GroupExtent e = group_extent(g, k, gy, gx);
  GroupDesc gd;
  int ident = 0;                                        // leading union entries whose token equals their position
  if (g.mode == kModeBand) {
    gd.n_union = band_union_keys(g, t.rad, e);
    const int nk = g.s[k] * g.s[k];
    for (int pt = 0; pt < band_parts(k); ++pt) {
      const BandPart b = band_part(g, t.rad, k, pt);
      const int glo = band_interval(b, nk, e.qy0).lo, ghi = band_interval(b, nk, e.qy1).hi;
      if (b.tok0 + glo != ident) break;
      ident += ghi - glo + 1;
      if (ghi != b.cols - 1) break;
    }
  } else {
    Box mine = {0, -1, 0, -1};
    if (lane <= k) mine = window_box(t.win, k, lane, e.qy0, e.qy1, e.qx0, e.qx1);
    int n = (mine.yhi - mine.ylo + 1) * (mine.xhi - mine.xlo + 1);
    gd.n_union = sum_of_lanes(n);
    // whole key scales from scale 0 on, then the first rows of the next box if it starts
    // at the scale's origin
    for (int j = 0; j <= k; ++j) {
      const Box b = {lane_value(mine.ylo, j), lane_value(mine.yhi, j), lane_value(mine.xlo, j), lane_value(mine.xhi, j)};
      const int gw = b.xhi - b.xlo + 1, rows = b.yhi - b.ylo + 1;
      if (b.ylo != 0 || b.xlo != 0 || g.off[j] != ident) break;
      if (gw != g.s[j]) { ident += gw; break; }
      ident += rows * gw;
      if (rows != g.s[j]) break;
    }
  }
  gd.union_base = 0;
  gd.n_phases = (gd.n_union + g.C - 1) / g.C;
  gd.k = k; gd.gy = gy; gd.gx = gx; gd.phase_base = 0;
  gd.ident = ident;
  return gd;
}

// K2: one wave per group of the list: the places of its patches, its key list and its phase tables, into their
// descriptors.  (first_ends carries the kept pairs to k_fill.)
template <class Count>
__global__ __launch_bounds__(64) void k_place(BlobPtrs p, PlaceList<kLaunchWords> s, int NW, int n_wide, int n_waves, int C) {
  const int lane = threadIdx.x, i = blockIdx.x, G = s.first_group + i, per = NW + n_wide;
  if (lane == 0) {
    GroupDesc& gd = p.groups[G];
    const int phase0 = (int)s.w[3 * i + 2];
    gd.union_base = phase0 * C; gd.n_phases = s.phases_of(i); gd.phase_base = phase0 * (n_wide ? n_wide : NW);
  }
  const Count own = lane < per ? s.template counts<Count>()[i * per + lane] : Count{0};
  int upto = own.steps();                               // steps of the patches up to the lane's
#pragma unroll
  for (int d = 1; d < 32; d <<= 1) { const int x = __shfl_up(upto, d); if (lane >= d) upto += x; }
  const int narrow = lane_value(upto, NW - 1);
  if (lane >= per) return;
  const bool wide = lane >= NW;
  WaveDesc& wd = p.waves[wide ? n_waves + G * n_wide + lane - NW : G * NW + lane];
  wd.step_begin = (int)s.w[3 * i + wide] + upto - own.steps() - (wide ? narrow : 0);
  wd.n_steps = own.steps();
  wd.first_ends = (uint32_t)own.pairs();
}

// the group's key list (token indices), padded to whole chunks with its last key; one wave
__device__ void fill_union(const Geom& g, const BlobPtrs& p, const Caps& caps, const GroupTables& t, const GroupDesc& gd) {
  const GroupExtent e = group_extent(g, gd.k, gd.gy, gd.gx);
  int32_t* out = p.union_tok + gd.union_base;
  if ((int64_t)gd.union_base + (int64_t)gd.n_phases * g.C > caps.n_union) return;
  int ubase = 0, last_tok = 0;
  if (g.mode == kModeBand) {
    const int nk = g.s[e.k] * g.s[e.k];
    for (int pt = 0; pt < band_parts(e.k); ++pt) {
      const BandPart b = band_part(g, t.rad, e.k, pt);
      const int glo = band_interval(b, nk, e.qy0).lo, ghi = band_interval(b, nk, e.qy1).hi;
      const int n = ghi - glo + 1;
      for (int i = threadIdx.x; i < n; i += blockDim.x) out[ubase + i] = b.tok0 + glo + i;
      ubase += n;
      last_tok = b.tok0 + ghi;
    }
  } else {
    __shared__ Box boxes[kMaxScales];                   // (the table is read once, by K threads at the same time)
    if ((int)threadIdx.x <= e.k) boxes[threadIdx.x] = window_box(t.win, e.k, (int)threadIdx.x, e.qy0, e.qy1, e.qx0, e.qx1);
    __syncthreads();
    for (int j = 0; j <= e.k; ++j) {
      const Box b = boxes[j];
      const int gw = b.xhi - b.xlo + 1, n = (b.yhi - b.ylo + 1) * gw;
      const bool dealt = g.n_wide > 0 && dealt_box(g.mode, ubase);
      for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const int row = i / gw;
        out[ubase + i] = g.off[j] + (b.ylo + (dealt ? dealt_row(row, b.yhi - b.ylo + 1) : row)) * g.s[j] + b.xlo + i - row * gw;
      }
      ubase += n;
      last_tok = g.off[j] + b.yhi * g.s[j] + b.xhi;
    }
  }
  for (int i = gd.n_union + threadIdx.x; i < gd.n_phases * g.C; i += blockDim.x) out[i] = last_tok;
}

// Step under construction: the wave's lanes deposit the keys they place (ring slot, token,
// query mask) in a 32-entry LDS buffer; when the step closes every lane picks the entries
// of its role in the attention kernel and the step is written with coalesced stores.
// Lane (n, g4) = (lane % 16, lane / 16):
//   K operand  rows of keys n and 16 + n          -> byte offset of its first 16-byte piece
//   V operand  rows of keys 4*g4 + n/4 (+16)      -> byte offset of its d-tile-0 8-byte read
//   mask bits  element e = 4*t + i  <->  key 16*t + 4*g4 + i against query n
struct StepBuf { uint32_t slot[kStepKeys]; int32_t tok[kStepKeys]; uint32_t qmask[kStepKeys]; };

//   Wide patches, lane (n, h) = (lane % 32, lane / 32):
//   K operand  row of key n                                                   -> byte offset of its 16-byte piece h
//   V operand  rows of keys 16*t + 8*j + 4*h + (lane % 16) / 4, t, j = 0, 1   -> byte offset of its read of dims 0..31
//   mask       key n against the patch's dimensions (see close)
template <bool WIDE>
struct FillSink {
  uint2* addr; uint64_t* mask; int32_t* toks; int32_t* phase_end;
  StepBuf* buf;
  int R, logC, lane;
  int n_steps, n_phases;               // what the plan has room for (the counts agree with the walk, or nothing beyond is written)
  int chunk = 0;                       // chunk of the last closed step: phase_end is written up to it
  int pairs = 0;                       // this lane's share of the kept pairs
  int ny = 0;                          // WIDE: of the patch (window mode), else 0
  int end0 = 0, end2 = 0;              // steps that end in chunk 0, in chunks 0 to 2
  // steps close in the order of their chunks, so the cumulative counts of the chunks that a step
  // skips are final when it closes: no counter is read back
  __device__ void fill_ends(int from, int to, int steps) {
    for (int i = from + lane; i < min(to, n_phases); i += 64) phase_end[i] = steps;
  }
  __device__ static uint32_t k_off(uint32_t slot, int g4) {
    return slot * kRingRowBytes + (((2u * g4) ^ ring_swizzle(slot)) << 4);
  }
  // wide patches: piece `piece` (0..3, of dims 0..31) of the row in `slot`
  __device__ static uint32_t piece_off(uint32_t slot, int piece) {
    return slot * kRingRowBytes + (((uint32_t)piece ^ ring_swizzle(slot)) << 4);
  }
  __device__ static uint32_t v_off(uint32_t slot, int n) {
    const uint32_t sw = ring_swizzle(slot), b = (n >> 1) & 1, half = n & 1;
    return slot * kRingRowBytes + 8u * half + 16u * ((b ^ sw) & 1u) + ((sw >> 1) << 5);
  }
  __device__ void keys(int, int idx, int upos, int t, unsigned qmask, bool take) {
    if (take) pairs += WIDE && ny > 0 ? __builtin_popcount(qmask & ((1u << ny) - 1u)) * __builtin_popcount(qmask >> ny) : __builtin_popcount(qmask);
    if (take) { buf->slot[idx] = (uint32_t)(upos % R); buf->tok[idx] = t; buf->qmask[idx] = qmask; }
  }
  __device__ void close(int step, int n_keys, int last_upos) {
    if (step >= n_steps) return;
    __syncthreads();                                   // (one wave per block) deposits are visible
    const int n = lane & 15, g4 = lane >> 4;
    const uint32_t pad = (uint32_t)(last_upos % R);    // padding keys read the step's last row
    auto slot_of = [&](int idx) { return idx < n_keys ? buf->slot[idx] : pad; };
    if constexpr (WIDE) {
      const int n5 = lane & 31, h = lane >> 5, l16 = lane & 15, piece = 2 * ((lane >> 4) & 1) + ((l16 & 3) >> 1);
      uint32_t v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = piece_off(slot_of(8 * i + 4 * h + (l16 >> 2)), piece) + 8u * (l16 & 1);
      // not kept by dimension i, i = 8 h + e (window mode: the query rows, then the query columns; bands: the queries)
      // -> bit 15 - 2 r of half e % 2, r = e / 2; bands: queries 16 + 8 h + e -> r + 4
      const uint32_t out = n5 < n_keys ? ~buf->qmask[n5] : ~0u;
      uint32_t m = 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        m |= ((out >> (8 * h + e)) & 1u) << (15 - 2 * (e >> 1) + 16 * (e & 1));
        m |= ((out >> (16 + 8 * h + e)) & 1u) << (7 - 2 * (e >> 1) + 16 * (e & 1));
      }
      ((uint4*)addr)[(int64_t)step * 64 + lane] = make_uint4(piece_off(slot_of(n5), h), v[0] | (v[1] << 16), v[2] | (v[3] << 16), m);
      end_step(step, last_upos);
      return;
    }
    if (addr) {
      const uint32_t k0 = k_off(slot_of(n), g4), k1 = k_off(slot_of(16 + n), g4);
      const uint32_t v0 = v_off(slot_of(4 * g4 + (n >> 2)), n), v1 = v_off(slot_of(16 + 4 * g4 + (n >> 2)), n);
      addr[(int64_t)step * 64 + lane] = make_uint2(k0 | (k1 << 16), v0 | (v1 << 16));
    }
    uint64_t mine = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int idx = 16 * (e >> 2) + 4 * g4 + (e & 3);
      const bool bit = idx < n_keys && ((buf->qmask[idx] >> n) & 1u);
      const uint64_t bal = __ballot(bit);
      if (lane == e) mine = bal;
    }
    if (lane < 8) mask[(int64_t)step * 8 + lane] = mine;
    if (lane < kStepKeys) toks[(int64_t)step * kStepKeys + lane] = lane < n_keys ? buf->tok[lane] : -1;
    if (addr) end_step(step, last_upos);
  }
  __device__ void end_step(int step, int last_upos) {
    const int c = last_upos >> logC;
    if (c > chunk) { fill_ends(chunk, c, step); chunk = c; }
    if (c == 0) end0 = step + 1;
    if (c <= 2) end2 = step + 1;
    __syncthreads();                                   // the buffer may be refilled
  }
};

// K3: one wave per (group, patch) and (group, wide patch): steps (ring addresses, lane masks, tokens) and the
// cumulative number of steps that are runnable after each phase; then one wave per group: its
// key list and descriptor (in the same launch: neither needs the other).  Bound: the serial walk of one wave.
// 480 patches of 30 head groups: 27 us, 35 us as two launches with counters that were read back; 30 us with the
// places in its arguments, where a count, a scan and it took 50 and the launches' gaps.  With the queries of a box's rows and
// columns found once per box, those of a band by bisection, and no wide patches in the kernel of plans without: 34 240 tokens
// 88 -> 68 us, a band over 2240 tokens 26 -> 20 (16 patches of 16 queries and 8 of 32 in a group).
// The descriptors and the header are written here.  With Places the places come with the arguments, else k_place has
// left them in the descriptors.  A patch whose walk ends at other counts than the host's, or a group of another number of
// phases, marks the header.
template <class PlacesArg, bool WIDE_PLAN>
__global__ __launch_bounds__(64) void k_fill(Geom g, BlobPtrs p, Caps caps, int n_waves, PlacesArg s) {
  constexpr bool PLACED = std::is_same_v<PlacesArg, Places>;
  __shared__ StepBuf buf;
  const int lane = threadIdx.x;
  const int n_wide = WIDE_PLAN ? caps.n_groups * kWidePatches : 0;
  const bool wide = WIDE_PLAN && (int)blockIdx.x >= n_waves, lists = (int)blockIdx.x >= n_waves + n_wide;
  const int idx = lists ? blockIdx.x - n_waves - n_wide : wide ? blockIdx.x - n_waves : blockIdx.x;
  const int per = lists ? 1 : wide ? kWidePatches : g.NW;
  const int G = idx / per, w = idx - G * per;
  const GroupTables t = group_tables(g, p, G);
  GroupDesc gd;
  int k, gy, gx;
  group_coords(g, t.grp, k, gy, gx);
  if constexpr (PLACED) {
    const int phase0 = (int)s.w[3 * G + 2];
    gd.n_phases = s.phases_of(G);
    gd.union_base = phase0 * g.C; gd.phase_base = phase0 * walked_patches(g);
  } else {
    const GroupDesc& placed = p.groups[G];
    gd.n_phases = placed.n_phases; gd.union_base = placed.union_base; gd.phase_base = placed.phase_base;
  }
  gd.k = k; gd.gy = gy; gd.gx = gx;
  if (lists) {
    GroupDesc own = group_desc(g, t, k, gy, gx, lane);
    if (own.n_phases != gd.n_phases) { p.hdr->error = kErrBuilder; return; }
    own.union_base = gd.union_base; own.phase_base = gd.phase_base;
    gd = own;
    if (lane == 0) p.groups[G] = gd;
    if (G == 0) {                                       // the header, but for the error that others may be marking
      Header h;
      memset(&h, 0, sizeof h);
      h.magic = kMagic; h.blob_bytes = caps.bytes;
      h.n_groups = caps.n_groups; h.n_waves = n_waves;
      h.n_steps = caps.n_steps; h.n_union = caps.n_union; h.n_phase_entries = caps.n_phase_entries;
      h.retained_pairs = caps.retained_pairs; h.n_wide_steps = caps.n_wide_steps;
      constexpr int kUsed = offsetof(Header, pad) / 4, kError = offsetof(Header, error) / 4;
#pragma unroll
      for (int i = 0; i < kUsed; ++i)
        if (i != kError && lane == 0) ((uint32_t*)p.hdr)[i] = ((const uint32_t*)&h)[i];
      if (lane >= kUsed) ((uint32_t*)p.hdr)[lane] = 0;
    }
    fill_union(g, p, caps, t, gd);
    return;
  }
  const GroupExtent e = group_extent(g, gd.k, gd.gy, gd.gx);
  const PatchExtent pe = wide ? wide_extent(g, gd.k, gd.gy, gd.gx, w) : patch_extent(g, gd.k, gd.gy, gd.gx, w);
  WaveDesc* const out = p.waves + blockIdx.x;
  WaveDesc wd = wide ? wide_desc(g, gd.k, pe) : patch_desc(g, gd.k, pe);
  int host_pairs;
  if constexpr (PLACED) {
    const int first = wide ? g.NW : 0;
    const SmallCount* counts = s.template counts<SmallCount>() + G * (g.NW + g.n_wide) + first;
    const SmallCount mine = counts[min(lane, w)], own = {(uint16_t)lane_value(mine.v, w)};
    wd.step_begin = (int)s.w[3 * G + wide] + sum_of_lanes(lane < w ? mine.steps() : 0);
    wd.n_steps = own.steps(); host_pairs = own.pairs();
  } else {
    wd.step_begin = out->step_begin; wd.n_steps = out->n_steps; host_pairs = (int)out->first_ends;
  }
  if ((int64_t)wd.step_begin + wd.n_steps > (wide ? caps.n_wide_steps : caps.n_steps) ||
      (int64_t)gd.phase_base + (int64_t)gd.n_phases * walked_patches(g) > caps.n_phase_entries) {
    p.hdr->error = kErrBuilder;
    return;
  }
  int ns, pairs = 0;
  uint32_t first_ends;
  auto fill = [&](auto& sink) {
    sink.buf = &buf; sink.R = g.R; sink.logC = g.logC; sink.lane = lane;
    sink.n_steps = wd.n_steps; sink.n_phases = gd.n_phases;
    sink.phase_end = p.phase_end + gd.phase_base + (int64_t)w * gd.n_phases;
  };
  if constexpr (WIDE_PLAN) if (wide) {
    FillSink<true> sink;
    fill(sink);
    sink.addr = (uint2*)((char*)p.step_addr + (int64_t)wd.step_begin * 64 * kWideDesc);
    sink.mask = nullptr; sink.toks = nullptr; sink.ny = g.mode == kModeBand ? 0 : pe.ny;
    ns = wave_walk_patch<true>(g, t.win, t.rad, e, pe, sink, lane);
    sink.fill_ends(sink.chunk, gd.n_phases, ns);
    first_ends = (uint32_t)sink.end0 | ((uint32_t)sink.end2 << 16);   // (a patch has at most 65535 steps)
    pairs = sum_of_lanes(sink.pairs);
  }
  if (!wide) {
    FillSink<false> sink;
    fill(sink);
    sink.addr = WIDE_PLAN ? nullptr : p.step_addr + (int64_t)wd.step_begin * 64;      // (wide patches: nobody walks the list in these steps)
    sink.mask = p.step_mask + (int64_t)wd.step_begin * 8;
    sink.toks = p.step_tok + (int64_t)wd.step_begin * kStepKeys;
    ns = wave_walk_patch<false>(g, t.win, t.rad, e, pe, sink, lane);
    if (sink.addr) sink.fill_ends(sink.chunk, gd.n_phases, ns);
    first_ends = (uint32_t)sink.end0 | ((uint32_t)sink.end2 << 16);
    pairs = sum_of_lanes(sink.pairs);
  }
  if (ns != wd.n_steps || pairs % kPairsModulus != host_pairs) { p.hdr->error = kErrBuilder; return; }
  if (!wide) wd.pairs = pairs;
  wd.first_ends = first_ends;
  if (lane == 0) *out = wd;
}

litevar_status build_plan(PlanSpec& sp, const PlanSizes& z, void* d_blob, hipStream_t st) {
  const Geom& g = sp.g;                  // (the host's part stays here)
  const BlobPtrs p = blob_ptrs(d_blob, z.off);
  Caps caps{z.n_steps, z.n_union, z.n_phase_entries, z.retained_pairs, z.n_wide_steps, z.bytes, g.n_groups * g.n_hg};
  const int ntab = g.mode == kModeWindow ? g.K * g.K * g.smax : g.K * g.K;
  const int tri = g.K * (g.K + 1) / 2, per_launch = kTableRadii / tri;
  TablesArg ta;
  ta.K = g.K; ta.mode = g.mode; ta.n_sink = g.n_sink; ta.smax = g.smax;
  for (int k = 0; k < g.K; ++k) ta.s[k] = (uint16_t)g.s[k];
  memcpy(ta.head_group, sp.head_group, sizeof ta.head_group);
  for (int hg0 = 0; hg0 < g.n_hg; hg0 += per_launch) {
    ta.hg0 = hg0; ta.n_hg = std::min(per_launch, g.n_hg - hg0); ta.n_heads = hg0 == 0 ? sp.n_heads : -1;
    int at = 0;
    for (int hg = hg0; hg < hg0 + ta.n_hg; ++hg)
      for (int k = 0; k < g.K; ++k)
        for (int j = 0; j <= k; ++j) ta.rad[at++] = sp.rad_all[((size_t)hg * g.K + k) * g.K + j];
    hipLaunchKernelGGL(k_tables, dim3((ntab + 255) / 256, ta.n_hg), dim3(256), 0, st, ta, p.win, p.rad, p.head_map, p.hdr);
  }
  const int n_all = g.n_groups * g.n_hg;
  const int nw = n_all * g.NW;
  const int n_wide = n_all * g.n_wide;
  const dim3 waves(nw + n_wide + n_all);
  bool small = true;
  for (const PlanSpec::PatchCount& c : sp.patch_counts) small = small && c.steps <= SmallCount::kMost;
  PlaceAt at;
  if (small && n_all <= groups_in<SmallCount>(kInlineWords, g.NW + g.n_wide)) {
    Places s;
    fill_list<SmallCount>(sp, 0, at, s);
    if (g.n_wide) hipLaunchKernelGGL((k_fill<Places, true>), waves, dim3(64), 0, st, g, p, caps, nw, s);
    else hipLaunchKernelGGL((k_fill<Places, false>), waves, dim3(64), 0, st, g, p, caps, nw, s);
  } else {
    PlaceList<kLaunchWords> s;
    for (int first = 0; first < n_all; first += s.n_groups) {
      if (small) fill_list<SmallCount>(sp, first, at, s);
      else fill_list<LargeCount>(sp, first, at, s);
      hipLaunchKernelGGL(small ? k_place<SmallCount> : k_place<LargeCount>, dim3(s.n_groups), dim3(64), 0, st, p, s, g.NW,
                         g.n_wide, nw, g.C);
    }
    if (g.n_wide) hipLaunchKernelGGL((k_fill<NoPlaces, true>), waves, dim3(64), 0, st, g, p, caps, nw, NoPlaces{});
    else hipLaunchKernelGGL((k_fill<NoPlaces, false>), waves, dim3(64), 0, st, g, p, caps, nw, NoPlaces{});
  }
  return hip_check(hipGetLastError(), "plan builder launch");
}

// ---- parity exports -------------------------------------------------------------

__global__ void k_export_win(int n, const int16_t* win, int16_t* out) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx < n) out[idx] = win[idx];
}

__global__ void k_fill_u8(uint8_t* p, size_t n, uint8_t v) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = v;
}

__global__ void k_zero_u64(unsigned long long* p) { if (threadIdx.x == 0 && blockIdx.x == 0) *p = 0; }

// local query row handled by column n of a patch, or -1
__device__ inline int patch_query_row(const WaveDesc& wd, int n) {
  return ((wd.valid >> n) & 1u) ? wd.q_base + (n / 4) * wd.sk + n % 4 : -1;
}

// one 64-lane block per (group, wave) of the head's group; lane (n, g4) owns the bits of
// query n for the keys {16t + 4*g4 + i} of every step
__global__ void k_export_dense(int L, const WaveDesc* waves, const int32_t* head_map, int head, int waves_per_hg,
                               const uint64_t* masks, const int32_t* toks, uint8_t* mask, unsigned long long* count) {
  const WaveDesc wd = waves[(size_t)head_map[head] * waves_per_hg + blockIdx.x];
  const int lane = threadIdx.x, n = lane % 16, g4 = lane / 16;
  const int qrow = patch_query_row(wd, n);
  unsigned long long local = 0;
  for (int s = 0; s < wd.n_steps; ++s) {
    const int64_t S = (int64_t)wd.step_begin + s;
    for (int e = 0; e < 8; ++e) {
      if (!(masks[S * 8 + e] >> lane & 1)) continue;
      const int tok = toks[S * kStepKeys + 16 * (e / 4) + 4 * g4 + e % 4];
      if (qrow >= 0 && tok >= 0) { mask[(size_t)qrow * L + tok] = 1; ++local; }
    }
  }
  if (count && local) atomicAdd(count, local);
}

__global__ void k_csr_count(const WaveDesc* waves, const int32_t* head_map, int head, int waves_per_hg,
                            const uint64_t* masks, int64_t* rowptr) {
  const WaveDesc wd = waves[(size_t)head_map[head] * waves_per_hg + blockIdx.x];
  const int lane = threadIdx.x, n = lane % 16;
  int cnt = 0;
  for (int s = 0; s < wd.n_steps; ++s)
    for (int e = 0; e < 8; ++e) cnt += (int)(masks[((int64_t)wd.step_begin + s) * 8 + e] >> lane & 1);
  cnt += __shfl_xor(cnt, 16); cnt += __shfl_xor(cnt, 32);
  const int qrow = patch_query_row(wd, n);
  if (lane < 16 && qrow >= 0) rowptr[qrow + 1] = cnt;
}

// in-place inclusive scan of rowptr[1..n] by one 1024-thread block
__global__ void k_csr_scan(int64_t* rowptr, int n) {
  __shared__ int64_t part[1024];
  const int t = threadIdx.x, per = (n + 1023) / 1024;
  const int b = t * per, e = b + per < n ? b + per : n;
  int64_t sum = 0;
  for (int i = b; i < e; ++i) sum += rowptr[i + 1];
  part[t] = sum;
  __syncthreads();
  if (t == 0) {
    int64_t acc = 0;
    for (int i = 0; i < 1024; ++i) { const int64_t v = part[i]; part[i] = acc; acc += v; }
    rowptr[0] = 0;
  }
  __syncthreads();
  int64_t acc = part[t];
  for (int i = b; i < e; ++i) { acc += rowptr[i + 1]; rowptr[i + 1] = acc; }
}

// 16 threads per patch, one per query: walk the steps in order and list the kept tokens
__global__ void k_csr_fill(const WaveDesc* waves, const int32_t* head_map, int head, int waves_per_hg,
                           const uint64_t* masks, const int32_t* toks, const int64_t* rowptr, int32_t* cols, int64_t cap) {
  const WaveDesc wd = waves[(size_t)head_map[head] * waves_per_hg + blockIdx.x];
  const int n = threadIdx.x;
  const int qrow = patch_query_row(wd, n);
  if (n >= 16 || qrow < 0) return;
  int64_t w = rowptr[qrow];
  const int64_t end = rowptr[qrow + 1];
  for (int s = 0; s < wd.n_steps; ++s) {
    const int64_t S = (int64_t)wd.step_begin + s;
    for (int idx = 0; idx < kStepKeys; ++idx) {
      const int r = idx % 16;
      if (masks[S * 8 + 4 * (idx / 16) + r % 4] >> ((r / 4) * 16 + n) & 1) {
        if (w < end && w < cap) cols[w] = toks[S * kStepKeys + idx];
        ++w;
      }
    }
  }
}

static int head_group_of(const litevar_plan* pl, int head) { return pl->n_heads > 0 ? pl->head_group[head] : 0; }

litevar_status export_window_table(const litevar_plan* pl, int head, int16_t* d_out, hipStream_t st) {
  const BlobPtrs p = blob_ptrs(pl->d_blob, pl->off);
  const int n = pl->n_scales * pl->n_scales * pl->side_max * 2;
  hipLaunchKernelGGL(k_export_win, dim3((n + 255) / 256), dim3(256), 0, st, n,
                     p.win + (size_t)head_group_of(pl, head) * n, d_out);
  return hip_check(hipGetLastError(), "window table export launch");
}

litevar_status export_dense(const litevar_plan* pl, int head, uint8_t* d_mask, uint64_t* d_count,
                            hipStream_t st) {
  const BlobPtrs p = blob_ptrs(pl->d_blob, pl->off);
  const size_t n = (size_t)pl->q_len * pl->kv_len;
  hipLaunchKernelGGL(k_fill_u8, dim3(2048), dim3(256), 0, st, d_mask, n, (uint8_t)0);
  if (d_count) hipLaunchKernelGGL(k_zero_u64, dim3(1), dim3(64), 0, st, (unsigned long long*)d_count);
  const int nw = pl->n_groups * pl->waves_per_group;
  hipLaunchKernelGGL(k_export_dense, dim3(nw), dim3(64), 0, st, pl->kv_len, p.waves, p.head_map, head, nw,
                     p.step_mask, p.step_tok, d_mask, (unsigned long long*)d_count);
  return hip_check(hipGetLastError(), "dense mask export launch");
}

litevar_status export_csr(const litevar_plan* pl, int head, int64_t* d_rowptr, int32_t* d_cols, size_t cap,
                          hipStream_t st) {
  const BlobPtrs p = blob_ptrs(pl->d_blob, pl->off);
  const int nw = pl->n_groups * pl->waves_per_group;
  hipLaunchKernelGGL(k_csr_count, dim3(nw), dim3(64), 0, st, p.waves, p.head_map, head, nw, p.step_mask, d_rowptr);
  hipLaunchKernelGGL(k_csr_scan, dim3(1), dim3(1024), 0, st, d_rowptr, pl->q_len);
  hipLaunchKernelGGL(k_csr_fill, dim3(nw), dim3(64), 0, st, p.waves, p.head_map, head, nw, p.step_mask, p.step_tok,
                     d_rowptr, d_cols, (int64_t)cap);
  return hip_check(hipGetLastError(), "csr export launch");
}

litevar_status read_header(const litevar_plan* pl, hipStream_t st, Header& h) {
  litevar_status rc = hip_check(hipStreamSynchronize(st), "hipStreamSynchronize");
  if (rc) return rc;
  return hip_check(hipMemcpy(&h, pl->d_blob, sizeof h, hipMemcpyDeviceToHost), "header copy");
}

}  // namespace lv
