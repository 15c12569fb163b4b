// bf16 attention forward for gfx950 (CDNA4) for plans that keep every pair of the block-causal
// map (radius -1, or windows that cover their parts): a query of scale k sees the tokens
// [0, off[k + 1]), so no work-list is needed and the queries are taken in token order.
//
// One workgroup = NWV waves of one (batch, head); a wave owns 32 consecutive query rows of one scale.
// The keys pass through LDS in chunks of 64 (K and V rows of 128 bytes, two buffers); the next
// chunk is requested into registers before the present one is computed and written to the other
// buffer after it, one barrier per chunk.  Per 32 keys:
//   S^T (32 keys x 32 queries) = K (A operand) . Q^T (B operand): v_mfma_f32_32x32x16_bf16; a
//       lane ends up with one query column and 16 of the 32 keys,
//   online softmax in base 2 with a lazily moved reference, as in the windowed kernels,
//   O^T (64 x queries) += V^T (A operand, ds_read_b64_tr_b16) . P^T (B operand: the lane's own
//       probabilities rounded to bf16; the key order of the slices is the order in which the score
//       tile's registers hold them), row sums of the rounded probabilities by v_dot2_f32_bf16.
// A wave's queries share their key limit; only the last block before it is masked.
//
// Why not the windowed kernels: a wave there issues 51 vector, 9 matrix and 12 LDS instructions (on such a
// plan) per 32 keys x 16 queries and fetches a step descriptor and lane masks; here 67, 8 and 13 serve 32
// queries (keys' rows on their way into LDS included), with nothing to fetch.  What bounds it now is the issue
// of vector and matrix instructions of one SIMD, which overlap little: at 2240 tokens and 288
// (batch, head) pairs the vector issue is busy 63 % of the cycles, the matrix pipe 44 %, the LDS pipe 39 %
// (windowed kernel on the same plan: 53, 28, 25).  119 and 127 registers (eight and four waves) let four waves
// share a SIMD.  Not faster, at that size: 64 queries per wave (342 us), the next chunk's
// score products issued between the exponentials, which takes 203 registers (365), chunks of 128
// keys (360), raised wave priority around the products (310, against 310 without).
// Measured against the windowed kernels (B H, tokens): 288, 2240: 427 -> 297 us (810 TFLOP/s of kept
// pairs); 480, 680: 117 -> 62 us; 2, 34 240: 6950 -> 500 us (the windowed kernel on one XCD per pair; 1820 spread).
#include <type_traits>

#include "attn_bf16_common.h"

namespace lv {

namespace {

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

constexpr int kChunk = 64;                     // keys per LDS buffer
constexpr int kRow = 128;                      // bytes of a K or V row

struct DenseArgs {
  AttnArgs a;
  uint32_t bh_magic;                           // floor(2^32 / (B H)), see divmod_by
  int q0, qb, qe;                              // token of query row 0; query scales [qb, qe)
  int n_units;                                 // of 32 rows of one scale
  int off[kMaxScales + 1];
  int unit_begin[kMaxScales + 1];              // units before scale k, k in [qb, qe)
};

// 16-byte piece p of row r is stored at piece position p ^ swizzle(r): eight consecutive rows put
// one piece into eight places (K reads), and four consecutive rows put a 32-byte unit into the four
// units of the row (the transposing V reads: 4 keys x 32 bytes per 16 lanes).
__device__ inline unsigned dense_swizzle(unsigned r) { return ((r & 3u) << 1) | ((r >> 2) & 1u); }

}  // namespace

// NWV = 8: two workgroups per CU, half the passes over K and V; NWV = 4: for launches that would not
// give every CU two of those.
template <int NWV>
__global__ __launch_bounds__(NWV * 64, 3)
void k_attn_bf16_dense(DenseArgs d, float c) {
  constexpr int kRowsAtOnce = NWV * 8;         // rows that the workgroup loads at once, eight lanes each
  constexpr int kRowsPerThread = kChunk / kRowsAtOnce;
  const AttnArgs& a = d.a;
  __shared__ __align__(1024) unsigned char Kbuf[2][kChunk * kRow], Vbuf[2][kChunk * kRow];

  // Tile by tile, the longest first, all (batch, head) pairs of one tile next to each other: the grid
  // ends on short tiles, and workgroup i runs on XCD i % 8, so that few pairs still use all XCDs.
  // (Measured against all tiles of a pair on one XCD: 2 pairs of 34 240 tokens 1660 -> 626 us, 288 of
  // 2240 tokens 324 -> 300 us, 480 of 680 tokens 73 -> 67 us, 16 of 34 240 tokens no change.)
  int tile, bh, b, h;
  divmod_by(a.first_block + blockIdx.x, (uint32_t)(a.B * a.H), d.bh_magic, tile, bh);
  divmod_by((uint32_t)bh, (uint32_t)a.H, a.H_magic, b, h);
  if (!plan_usable(a.hdr)) return;

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int n = lane & 31, hh = lane >> 5;
  // Units of 32 rows of one scale (the last one of a scale may be short), tiles of NWV units laid from
  // the last unit backwards: the longest tiles start first and are full.
  struct Unit { int k, rows_before; };         // query scale, rows of the scale before the unit
  // (lane k holds scale k's numbers and a ballot finds the scale; a loop over the kernel's arguments is a scalar
  // round trip per scale: 30 scales of one row, 32 pairs 7.8 -> 4.6 us, 480 pairs 25.6 -> 16.3)
  const int my_off = d.off[min(lane, kMaxScales)], my_begin = d.unit_begin[min(lane, kMaxScales)];
  auto off = [&](int k) -> int { return __builtin_amdgcn_readlane(my_off, k); };
  auto unit_at = [&](int u) -> Unit {          // (units below 0: the first)
    u = max(u, 0);
    const int k = d.qb + __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane >= d.qb && lane < d.qe && my_begin <= u)) - 1;
    return Unit{k, 32 * (u - __builtin_amdgcn_readlane(my_begin, k))};
  };
  const int tile_end = d.n_units - tile * NWV;           // unit behind the tile's last
  const int k_last = unit_at(tile_end - 1).k;
  const int unit = tile_end - NWV + wave;
  const Unit un = unit_at(unit);
  auto is_shared = [&](int k) -> bool { return a.cfg_share && a.cfg_share[h * a.n_scales + k]; };
  const bool partner = a.cfg_share && b >= a.B / 2;      // an unconditional row of a call with sharing
  if (partner) {                               // all rows written by the conditional workgroup?
    bool all = true;
    for (int k = unit_at(tile_end - NWV).k; k <= k_last; ++k) all = all && is_shared(k);
    if (all) return;
  }
  const int n_keys = off(k_last + 1);                                // keys of the tile
  const int wave_keys = unit < 0 ? 0 : off(un.k + 1);                // keys that the wave's queries see
  const int scale_rows = off(un.k + 1) - off(un.k);
  const int row = off(un.k) - d.q0 + un.rows_before + n;
  const bool row_ok = unit >= 0 && un.rows_before + n < scale_rows;

  // Q^T as the B operand: lane (n, hh) holds Q[query n][16 t + 8 hh .. + 7]
  bf16x8 qf[4];
  {
    // (a lane without a query holds some other one; it is not stored)
    const int r = row_ok ? checked_index(a.hdr, row, a.q_len) : min(row, a.q_len - 1);
    const __bf16* qp = (const __bf16*)a.q + b * a.qs[0] + h * a.qs[1] + r * a.qs[2] + 8 * hh;
#pragma unroll
    for (int t = 0; t < 4; ++t) qf[t] = as_bf16x8(*(const uint4*)(qp + 16 * t));
  }

  // loading duty: piece tid % 8 of rows tid / 8 + kRowsAtOnce i of every chunk (keys past the last are
  // read from the last row: always in bounds, masked)
  const unsigned char* Kp = (const unsigned char*)((const __bf16*)a.k + b * a.ks[0] + h * a.ks[1]) + 16 * (tid & 7);
  const unsigned char* Vp = (const unsigned char*)((const __bf16*)a.v + b * a.ks[0] + h * a.ks[1]) + 16 * (tid & 7);
  const unsigned row_bytes = (unsigned)a.ks[2] * 2u;     // (a slab spans < 2 GiB, checked by the API)
  const int lrow = tid >> 3;
  const unsigned lds_dst = (unsigned)lrow * kRow + ((((unsigned)tid & 7u) ^ dense_swizzle((unsigned)lrow)) << 4);
  auto load_rows = [&](const unsigned char* p, int key0, u32x4 (&r)[kRowsPerThread]) {
#pragma unroll
    for (int i = 0; i < kRowsPerThread; ++i)
      r[i] = *(const u32x4*)(p + __umul24((unsigned)checked_index(a.hdr, min(key0 + lrow + kRowsAtOnce * i, n_keys - 1), a.kv_len),
                                          row_bytes));
  };
  auto store_rows = [&](unsigned char* buf, const u32x4 (&r)[kRowsPerThread]) {
#pragma unroll
    for (int i = 0; i < kRowsPerThread; ++i)   // (32 or 64 rows on, the swizzle is the same)
      *(u32x4*)(buf + lds_dst + kRowsAtOnce * kRow * i) = r[i];
  };

  // LDS read offsets: K piece 2 t + hh of row n; V: 4 keys x 16 dims per 16 lanes
  unsigned k_off[4], v_off[2];
#pragma unroll
  for (int t = 0; t < 4; ++t) k_off[t] = (unsigned)n * kRow + ((((unsigned)(2 * t + hh)) ^ dense_swizzle((unsigned)n)) << 4);
#pragma unroll
  for (int dt = 0; dt < 2; ++dt) {
    const unsigned l16 = (unsigned)lane & 15u, r = 4u * (unsigned)hh + (l16 >> 2);
    const unsigned piece = 4u * dt + 2u * (((unsigned)lane >> 4) & 1u) + ((l16 & 3u) >> 1);
    v_off[dt] = r * kRow + ((piece ^ dense_swizzle(r)) << 4) + 8u * (l16 & 1u);
  }

  f32x16 O[2] = {f32x16{}, f32x16{}};
  float L = 0.f, negmc = 0.f, thr = kFloor;    // row sum of this lane's keys, -m c, and the score above which m moves
  const float slack = kSlack / c;
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};

  // 32 keys against the wave's 32 queries (K, V: their rows in LDS)
  auto run_block = [&](const unsigned char* K, const unsigned char* V, int key0) {
    f32x16 S = f32x16{};
#pragma unroll
    for (int t = 0; t < 4; ++t)
      S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(*(const uint4*)(K + k_off[t])), qf[t], S, 0, 0, 0);
    s16x4 va[2][2][2];                         // [slice of 16 keys][dim tile][half]
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int j = 0; j < 2; ++j) va[t][dt][j] = lds_read_tr16(V + v_off[dt] + (16 * t + 8 * j) * kRow);
    if (key0 + 32 > wave_keys) {               // (uniform)
      // keys of later scales: no score, and V rows of zeros (whatever they hold must not reach the sums)
      const int left = wave_keys - key0 - 4 * hh;
#pragma unroll
      for (int e = 0; e < 16; ++e)
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
          va[e >> 3][dt][(e >> 2) & 1][e & 3] = 8 * (e >> 2) + (e & 3) < left ? va[e >> 3][dt][(e >> 2) & 1][e & 3] : (short)0;
#pragma unroll
      for (int e = 0; e < 16; ++e) S[e] = 8 * (e >> 2) + (e & 3) < left ? S[e] : -INFINITY;
    }
    float mx = S[0], my = S[1];
#pragma unroll
    for (int e = 2; e < 14; e += 4) { mx = fmaxf(fmaxf(mx, S[e]), S[e + 1]); my = fmaxf(fmaxf(my, S[e + 2]), S[e + 3]); }
    mx = fmaxf(fmaxf(mx, S[14]), S[15]);
    mx = fmaxf(mx, my);
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(mx > thr) != 0, 0)) {   // rare after the first blocks
      const unsigned u = __float_as_uint(mx);
      auto sw = __builtin_amdgcn_permlane32_swap(u, u, false, false);
      const unsigned s0 = sw[0], s1 = sw[1];
      const float mxr = fmaxf(__uint_as_float(s0), __uint_as_float(s1));   // over both lanes of the query
      if (mxr > thr) {
        const float nmc = -mxr * c;
        const float alpha = thr == kFloor ? 1.f : __builtin_amdgcn_exp2f(nmc - negmc);   // (while m is unset the sums are zero)
        negmc = nmc; thr = mxr + slack;
        L *= alpha; O[0] *= alpha; O[1] *= alpha;
      }
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      bf16x8 pb;
#pragma unroll
      for (int e = 0; e < 8; ++e) pb[e] = (__bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(S[8 * t + e], c, negmc));
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        const bf16x2 two = {pb[e], pb[e + 1]};
        L = __builtin_amdgcn_fdot2_f32_bf16(two, ones, L, false);
      }
#pragma unroll
      for (int dt = 0; dt < 2; ++dt) {
        const s16x8 v8 = {va[t][dt][0][0], va[t][dt][0][1], va[t][dt][0][2], va[t][dt][0][3],
                          va[t][dt][1][0], va[t][dt][1][1], va[t][dt][1][2], va[t][dt][1][3]};
        O[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, v8), pb, O[dt], 0, 0, 0);
      }
    }
  };
  u32x4 kr[kRowsPerThread], vr[kRowsPerThread];
  load_rows(Kp, 0, kr); load_rows(Vp, 0, vr);
  store_rows(Kbuf[0], kr); store_rows(Vbuf[0], vr);
  // (the queries' registers are tied to this point: a wait for them inside the loop would also wait
  // for the chunk that has just been requested)
  asm volatile("" : "+v"(qf[0]), "+v"(qf[1]), "+v"(qf[2]), "+v"(qf[3]));
  __syncthreads();
  auto one = [&](int key0, auto odd) {
    constexpr int p = decltype(odd)::value;
    const bool more = key0 + kChunk < n_keys;
    if (more) { load_rows(Kp, key0 + kChunk, kr); load_rows(Vp, key0 + kChunk, vr); }
#pragma unroll
    for (int blk = 0; blk < kChunk / 32; ++blk) {
      if (key0 + 32 * blk < wave_keys) run_block(Kbuf[p] + blk * 32 * kRow, Vbuf[p] + blk * 32 * kRow, key0 + blk * 32);
    }
    if (more) { store_rows(Kbuf[p ^ 1], kr); store_rows(Vbuf[p ^ 1], vr); }   // (read last in the chunk before)
    __syncthreads();
  };
  for (int key0 = 0; key0 < n_keys; key0 += 2 * kChunk) {
    one(key0, std::integral_constant<int, 0>{});
    if (key0 + kChunk < n_keys) one(key0 + kChunk, std::integral_constant<int, 1>{});
  }

  const unsigned u = __float_as_uint(L);
  auto sw = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const unsigned s0 = sw[0], s1 = sw[1];
  const float inv = 1.f / (__uint_as_float(s0) + __uint_as_float(s1));
  if (!row_ok) return;
  const bool shared = is_shared(un.k);
  if (shared && partner) return;               // the conditional workgroup writes this row
  __bf16* op = (__bf16*)a.o + b * a.os[0] + h * a.os[1] + checked_index(a.hdr, row, a.q_len) * a.os[2] + 4 * hh;
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      bf16x4 r;
#pragma unroll
      for (int i = 0; i < 4; ++i) r[i] = (__bf16)(O[dt][4 * j + i] * inv);
      *(bf16x4*)(op + 32 * dt + 8 * j) = r;
      if (shared) *(bf16x4*)(op + (a.B / 2) * a.os[0] + 32 * dt + 8 * j) = r;
    }
}

// Plans that keep every pair of the block-causal map, however their radii say so, go to the kernel
// above, unless the plan asks for a shape of the windowed kernels (waves_per_group and the like).  Up to
// 16 rows -- one patch -- the four- and eight-patch kernel is as fast: (B H, rows), windowed / dense:
// 480, 9: 4.6 / 5.0 us; 480, 25: 5.7 / 5.1; 480, 30: 9.8 / 5.8; 8, 64: 6.8 / 6.7; 4, 256: 16.5 / 13.9.
// So it is, or faster, while the windowed workgroups are about two per CU or fewer and their patches take
// few steps.  Workgroups x steps per patch: 120 x 4 scales 1 2 3 4, 480 x 1: 4.0 / 4.4 us; 480 x 4, 1920 x 1: 9.3 /
// 5.2; scales 1 to 6, 192 x 2: 5.1 / 5.7, 720 x 2: 7.4 / 5.8; ten of side 4, 80 x 3: 5.9 / 6.5, 1200 x 3: 10.4 / 6.8; three
// of side 6, 96 x 3: 5.7 / 5.8, 360 x 3: 6.6 / 5.9; one of 12 x 12, 24 x 6: 6.8 / 6.9; one of 13 x 13, 32 x 14: 11.5 / 10.2.
bool takes_dense_kernel(const litevar_plan* pl, int64_t bh) {
  if (pl->q_len <= kPatchQueries || pl->tiling_chosen || pl->patches_per_wave != 0 || pl->spin_limit != kDefaultSpinLimit)
    return false;
  const int64_t patches = (int64_t)pl->n_patches * pl->n_head_groups;
  if (pl->n_steps <= 3 * patches && (pl->n_steps < 1 || bh * pl->n_groups <= 512 * patches / pl->n_steps)) return false;
  int64_t off = 0, all = 0;
  for (int k = 0; k < pl->q_scale_end; ++k) {
    const int64_t n = (int64_t)pl->scales[k] * pl->scales[k];
    off += n;
    if (k >= pl->q_scale_begin) all += n * off;
  }
  for (int i = 0; i < pl->n_head_groups; ++i)
    if (pl->retained_pairs_of_group[i] != all) return false;
  return true;
}

litevar_status launch_attn_bf16_dense(const litevar_plan* pl, const AttnArgs& a, hipStream_t st) {
  DenseArgs d{};
  d.a = a;
  d.off[0] = 0;
  for (int k = 0; k < pl->n_scales; ++k) d.off[k + 1] = d.off[k] + pl->scales[k] * pl->scales[k];
  d.n_units = 0;
  for (int k = 0; k <= pl->n_scales; ++k) {
    d.unit_begin[k] = d.n_units;
    if (k >= pl->q_scale_begin && k < pl->q_scale_end) d.n_units += (d.off[k + 1] - d.off[k] + 31) / 32;
  }
  d.q0 = pl->q_token_begin; d.qb = pl->q_scale_begin; d.qe = pl->q_scale_end;
  // Eight waves (256 rows) per workgroup once the rows would fill 300 such workgroups, with fewer of
  // them CUs stand idle.  (B H, rows), four / eight waves: 2, 34 240 (268 workgroups' worth): 496 / 611 us;
  // 480, 100 (188): 11.0 / 11.7; 32, 680 (85): 14.3 / 18.6; 480, 169 (317): 22.8 / 21.6; 480, 256 (480):
  // 35.2 / 33.1; 60, 2240 (525): 64.6 / 60.8.  With fewer rows where eight waves take all units of a pair and four
  // would pass twice over many keys.  480 pairs, 144 rows: 4240 keys 160 / 136; 1168: 42.0 / 39.3; 169: 11.8 / 12.4.
  const int64_t BH = (int64_t)a.B * a.H;
  const bool one_pass = d.n_units > 4 && d.n_units <= 8 && BH >= 300 && d.off[d.qe] >= 1024;
  const int nwv = BH * a.q_len >= 300 * 256 || one_pass ? 8 : 4;
  const int64_t blocks = BH * ((d.n_units + nwv - 1) / nwv);
  if (blocks > 0x7fffffff) return fail(LITEVAR_E_UNSUPPORTED, "grid too large");
  d.bh_magic = (uint32_t)(((uint64_t)1 << 32) / (uint64_t)BH - (BH <= 1));
  const float c = a.sm_scale * 1.4426950408889634f;
  return launch_in_parts(blocks, nwv * 64, "dense bf16 attention launch", [&](int64_t first, unsigned n) {
    d.a.first_block = (uint32_t)first;
    if (nwv == 8) hipLaunchKernelGGL(k_attn_bf16_dense<8>, dim3(n), dim3(nwv * 64), 0, st, d, c);
    else hipLaunchKernelGGL(k_attn_bf16_dense<4>, dim3(n), dim3(nwv * 64), 0, st, d, c);
  });
}

}  // namespace lv
