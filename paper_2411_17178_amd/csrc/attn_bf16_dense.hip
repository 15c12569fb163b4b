// bf16 attention forward for gfx950 (CDNA4) for plans that keep every pair of the block-causal
// map (radius -1, or windows that cover their parts): a query of scale k sees the tokens
// [0, off[k + 1]), so no work-list is needed and the queries are taken in token order.
//
// One workgroup = NWV waves of one (batch, head); a wave owns 32 consecutive query rows of one scale.
// The keys pass through LDS in chunks of 64 (K and V rows of 128 bytes, two or three buffers), which LDS-DMA transfers
// fill while the chunk before is computed.  Per 32 keys:
//   S^T (32 keys x 32 queries) = K (A operand) . Q^T (B operand): v_mfma_f32_32x32x16_bf16; a
//       lane ends up with one query column and 16 of the 32 keys,
//   softmax in base 2 with the first block's largest score as the reference, which moves only when a row sum passes 2^40,
//   O^T (64 x queries) += V^T (A operand, ds_read_b64_tr_b16) . P^T (B operand: the lane's own
//       probabilities rounded to bf16; the key order of the slices is the order in which the score
//       tile's registers hold them), row sums of the rounded probabilities by v_dot2_f32_bf16, one chain per slice.
// The score products of a block are issued before the exponentials of the block before it, so that the matrix pipe works
// under them.  A wave's queries share their key limit; only the last block before it is masked.
//
// Why not the windowed kernels: their steps fetch descriptors and masks; here 61 vector, 8 matrix and 12 LDS instructions
// serve 32 keys x 32 queries, with nothing to fetch.  At 2240 tokens and 288 (batch, head) pairs the vector issue is
// busy 67 % of the cycles and the matrix pipe 48 % (with the maximum of the scores, transfers through registers and no
// products ahead: 63 and 44 %, 297 us; now 275 us, 875 TFLOP/s of kept pairs), but the clock falls to 1.7 GHz under it
// (1.8 before): what bounds it is the power that the instructions take, more than their number per cycle.  127 registers let
// four waves share a SIMD.  One chain of row sums: 280 us.  Not faster in the kernel before: 64 queries per wave
// (342 us), chunks of 128 keys (360), raised wave priority around the products (310, against 310 without).
// Before / now (B H, tokens): 480, 680: 62.5 / 57.7 us; 32, 680: 14.3 / 13.1; 2, 34 240: 513 / 476; 8, 256 queries on 680: 14.0 / 12.8.
#include <type_traits>

#include "attn_bf16_common.h"

namespace lv {

namespace {

constexpr int kChunk = 64;                     // keys per LDS buffer
constexpr int kRow = 128;                      // bytes of a K or V row
constexpr int kBufBytes = 2 * kChunk * kRow;   // K rows, V rows

// the keys [0, n) for attend_row
struct AllKeys {
  int n, n_blocks;
  __device__ bool key(int block, int i, int& tok) const { tok = min(32 * block + i, n - 1); return 32 * block + i < n; }
};

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

// K rows of a block as the A operand and its V rows, transposed: va[4 t + 2 j + dt], slice t of 16 keys, its half j, head
// dimension tile dt.  Issued only; a wait must precede the first use.  AT: byte offset of the block's rows.
template <int AT>
__device__ inline void read_k(const unsigned (&k)[4], u32x4 (&r)[4]) {
  asm volatile("ds_read_b128 %0, %4 offset:%8\n\tds_read_b128 %1, %5 offset:%8\n\t"
               "ds_read_b128 %2, %6 offset:%8\n\tds_read_b128 %3, %7 offset:%8"
               : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3])
               : "v"(k[0]), "v"(k[1]), "v"(k[2]), "v"(k[3]), "i"(AT) : "memory");
}
template <int AT>
__device__ inline void read_v(const unsigned (&v)[2], u32x2 (&va)[8]) {
  asm volatile("ds_read_b64_tr_b16 %0, %8 offset:%10\n\tds_read_b64_tr_b16 %1, %9 offset:%10\n\t"
               "ds_read_b64_tr_b16 %2, %8 offset:%11\n\tds_read_b64_tr_b16 %3, %9 offset:%11\n\t"
               "ds_read_b64_tr_b16 %4, %8 offset:%12\n\tds_read_b64_tr_b16 %5, %9 offset:%12\n\t"
               "ds_read_b64_tr_b16 %6, %8 offset:%13\n\tds_read_b64_tr_b16 %7, %9 offset:%13"
               : "=&v"(va[0]), "=&v"(va[1]), "=&v"(va[2]), "=&v"(va[3]),
                 "=&v"(va[4]), "=&v"(va[5]), "=&v"(va[6]), "=&v"(va[7])
               : "v"(v[0]), "v"(v[1]), "i"(AT), "i"(AT + 8 * kRow), "i"(AT + 16 * kRow), "i"(AT + 24 * kRow) : "memory");
}

}  // namespace

// NWV = 8: half the passes over K and V; NWV = 4: for launches that would not fill the chip with those.
// BUFS = 3: one chunk being read, one landing, one whose last readers may be behind, one barrier per chunk; BUFS = 2: a
// second barrier, behind which the chunk that has just been read is replaced; four workgroups of four waves then share a
// CU instead of three.
template <int NWV, int BUFS>
__global__ __launch_bounds__(NWV * 64) __attribute__((amdgpu_waves_per_eu(NWV == 4 && BUFS == 3 ? 3 : 4, NWV == 4 && BUFS == 3 ? 3 : 4)))
void k_attn_bf16_dense(DenseArgs d, float c) {
  constexpr int kRowsPerWave = kChunk / NWV, kTransfers = kRowsPerWave / 8;   // per chunk; a transfer is 8 rows, eight lanes each
  const AttnArgs& a = d.a;
  __shared__ __align__(1024) unsigned char smem[BUFS * kBufBytes];

  // Tile by tile, the longest first, all (batch, head) pairs of one tile next to each other: the grid
  // ends on short tiles, and workgroup i runs on XCD i % 8, so that few pairs still use all XCDs.
  // (Measured against all tiles of a pair on one XCD: 2 pairs of 34 240 tokens 1660 -> 626 us, 288 of
  // 2240 tokens 324 -> 300 us, 480 of 680 tokens 73 -> 67 us, 16 of 34 240 tokens no change.)
  int tile, bh, b, h;
  divmod_by(a.first_block + blockIdx.x, (uint32_t)(a.B * a.H), d.bh_magic, tile, bh);
  divmod_by((uint32_t)bh, (uint32_t)a.H, a.H_magic, b, h);
  if (!plan_usable(a.hdr)) return;
  asm volatile("" : "+s"(c));                // (so that no block waits for it)

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

  // loading duty: rows kRowsPerWave wave .. of every chunk, lane l piece l % 8 of row l / 8 of a transfer, put where the
  // swizzle wants it by choosing the piece that is fetched (keys past the last are read from the last row: always in
  // bounds, masked)
  const unsigned char* Kp = (const unsigned char*)((const __bf16*)a.k + b * a.ks[0] + h * a.ks[1]);
  const unsigned char* Vp = (const unsigned char*)((const __bf16*)a.v + b * a.ks[0] + h * a.ks[1]);
  const unsigned row_bytes = (unsigned)a.ks[2] * 2u;     // (a slab spans < 2 GiB, checked by the API)
  const int lrow = lane >> 3;
  const unsigned piece_off = (((unsigned)lane & 7u) ^ dense_swizzle((unsigned)lrow)) << 4;
  auto issue_chunk = [&](int chunk, int buf) {
#pragma unroll
    for (int i = 0; i < kTransfers; ++i) {
      const int row0 = kRowsPerWave * wave + 8 * i, key = min(kChunk * chunk + row0 + lrow, n_keys - 1);
      const unsigned src = __umul24((unsigned)checked_index(a.hdr, key, a.kv_len), row_bytes) + piece_off;
      unsigned char* dst = smem + buf * kBufBytes + row0 * kRow;
      __builtin_amdgcn_global_load_lds((global_void*)(Kp + src), (lds_void*)dst, 16, 0, 0);
      __builtin_amdgcn_global_load_lds((global_void*)(Vp + src), (lds_void*)(dst + kChunk * kRow), 16, 0, 0);
    }
  };

  // LDS read offsets: K piece 2 t + hh of row n; V: 4 keys x 16 dims per 16 lanes
  unsigned k_off[4], v_off[2];
#pragma unroll
  for (int t = 0; t < 4; ++t)
    k_off[t] = lds_addr(smem) + (unsigned)n * kRow + ((((unsigned)(2 * t + hh)) ^ dense_swizzle((unsigned)n)) << 4);
#pragma unroll
  for (int dt = 0; dt < 2; ++dt) {
    const unsigned l16 = (unsigned)lane & 15u, r = 4u * (unsigned)hh + (l16 >> 2);
    const unsigned piece = 4u * dt + 2u * (((unsigned)lane >> 4) & 1u) + ((l16 & 3u) >> 1);
    v_off[dt] = lds_addr(smem) + r * kRow + ((piece ^ dense_swizzle(r)) << 4) + 8u * (l16 & 1u);
  }

  f32x16 O[2] = {f32x16{}, f32x16{}};
  float L[2] = {0.f, 0.f}, negm = 0.f;         // this lane's part of the row sum, one chain per slice; minus the softmax reference (base 2)
  const uint64_t queries = __builtin_amdgcn_ballot_w64(row_ok);
  uint64_t unset = queries;                    // lanes whose query has no reference yet
  uint64_t moved = 0;                          // lanes whose reference has moved
  uint64_t far = 0;                            // lanes whose reference was beyond kFarReference at some time

  // S^T of a block whose K rows have been requested
  auto scores = [&](u32x4 (&kr)[4]) -> f32x16 {
    lds_wait_k(kr[0], kr[1], kr[2], kr[3]);
    f32x16 S = f32x16{};
#pragma unroll
    for (int t = 0; t < 4; ++t)
      S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kr[t]), qf[t], S, 0, 0, 0);
    return S;
  };
  // The rest of a block, its V rows requested.  The softmax reference is the largest score of the first block (so that few
  // keys give the bits that the windowed kernels give) and moves only when a query's sum passes 2^40.
  auto absorb = [&](f32x16& S, u32x2 (&va)[8], int key0) {
    if (key0 + 32 > wave_keys) {               // (uniform)
      // keys of later scales: no score, and V rows of zeros (whatever they hold must not reach the sums)
      const int left = wave_keys - key0 - 4 * hh;
      lds_wait_v_wide(va);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int first = left - 8 * (i >> 1);           // of the four keys of va[i]: that many are the wave's
        va[i].x &= first > 1 ? ~0u : first > 0 ? 0xffffu : 0u;
        va[i].y &= first > 3 ? ~0u : first > 2 ? 0xffffu : 0u;
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) S[e] = 8 * (e >> 2) + (e & 3) < left ? S[e] : -INFINITY;
    }
    auto largest = [&]() {                     // score of the query, over both of its lanes
      float mx = S[0];
#pragma unroll
      for (int e = 1; e < 16; ++e) mx = fmaxf(mx, S[e]);
      return fmaxf(mx, other_half(mx));
    };
    if (__builtin_expect(unset != 0, 0)) {
      const float mx = largest();
      const bool set = __builtin_amdgcn_inverse_ballot_w64(unset) && mx > kFloor;
      negm = set ? -mx * c : negm;
      unset &= ~__builtin_amdgcn_ballot_w64(set);
      far |= is_far(negm);
    }
    bf16x8 pb[2];
    float sum[2];
    auto exponentials = [&]() {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        sum[t] = L[t];
#pragma unroll
        for (int e = 0; e < 8; ++e) pb[t][e] = (__bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(S[8 * t + e], c, negm));
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
          const bf16x2 two = {pb[t][e], pb[t][e + 1]};
          sum[t] = __builtin_amdgcn_fdot2_f32_bf16(two, kOnes, sum[t], false);
        }
      }
    };
    exponentials();
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(fmaxf(sum[0], sum[1]) > kMostSum) != 0, 0)) {
      auto both = [&](const float (&x)[2]) { const float y = x[0] + x[1]; return y + other_half(y); };   // slices, lanes
      const float mx = largest(), now = both(sum), before = both(L);
      float to = mx > kFloor ? __builtin_fmaf(mx, c, negm) : kFloor;
      if (before > 0.f) to = fmaxf(to, __builtin_amdgcn_logf(before));         // (base 2)
      const float shift = now > kMostSum && to > kFloor ? rintf(to) : 0.f;
      const float alpha = before > 0.f ? __builtin_amdgcn_exp2f(-shift) : 1.f;
      negm -= shift; L[0] *= alpha; L[1] *= alpha;
      far |= is_far(negm);
      moved |= __builtin_amdgcn_ballot_w64(shift != 0.f);
#pragma unroll
      for (int e = 0; e < 16; ++e) { O[0][e] *= alpha; O[1][e] *= alpha; }
      exponentials();
    }
    L[0] = sum[0]; L[1] = sum[1];
    lds_wait_v_wide(va);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int dt = 0; dt < 2; ++dt) {
        const uint4 v8 = {va[4 * t + dt].x, va[4 * t + dt].y, va[4 * t + 2 + dt].x, va[4 * t + 2 + dt].y};
        O[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(v8), pb[t], O[dt], 0, 0, 0);
      }
  };

  const int n_chunks = (n_keys + kChunk - 1) / kChunk;
  issue_chunk(0, 0);
  if (n_chunks > 1) { issue_chunk(1, 1); wait_vmcnt<2 * kTransfers>(); } else wait_vmcnt<0>();
  asm volatile("" : "+v"(qf[0]), "+v"(qf[1]), "+v"(qf[2]), "+v"(qf[3]));   // (older than the chunks: in)
  asm volatile("s_barrier" ::: "memory");
  f32x16 S0 = f32x16{};                        // scores of the chunk's first block
  if (wave_keys > 0) {
    u32x4 kr[4];
    read_k<0>(k_off, kr);
    S0 = scores(kr);
  }
  // A chunk: its two blocks, each with the next block's score products in front of its own exponentials, which then
  // run under them.  Between the blocks the next chunk is waited for -- the only transfers in flight -- and the
  // one after it is requested, into the buffer that every wave has read to its end by then.
  auto one = [&](int chunk, auto which) -> bool {
    constexpr int p = decltype(which)::value, AT = p * kBufBytes, NEXT = (p + 1) % BUFS * kBufBytes;
    const int key0 = chunk * kChunk;
    const bool more = chunk + 1 < n_chunks;
    f32x16 S1;
    asm volatile("" : "=v"(S1));            // (not set where the wave has no second block, and not used then)
    if (key0 < wave_keys) {
      u32x2 va[8];
      if (key0 + 32 < wave_keys) {
        u32x4 kr[4];
        read_k<AT + 32 * kRow>(k_off, kr);
        S1 = scores(kr);
      }
      read_v<AT + kChunk * kRow>(v_off, va);
      __builtin_amdgcn_sched_barrier(0);
      absorb(S0, va, key0);
    }
    if (more) {
      wait_vmcnt<0>();
      asm volatile("s_barrier" ::: "memory");
      if (BUFS == 3 && chunk + 2 < n_chunks) issue_chunk(chunk + 2, (p + 2) % BUFS);
    }
    if (key0 + 32 < wave_keys) {
      u32x2 va[8];
      if (key0 + kChunk < wave_keys) {
        u32x4 kr[4];
        read_k<NEXT>(k_off, kr);
        S0 = scores(kr);
      }
      read_v<AT + (kChunk + 32) * kRow>(v_off, va);
      __builtin_amdgcn_sched_barrier(0);
      absorb(S1, va, key0 + 32);
    }
    if (BUFS == 2 && chunk + 2 < n_chunks) {
      asm volatile("s_barrier" ::: "memory");
      issue_chunk(chunk + 2, p);
    }
    return more;
  };
  for (int chunk = 0;; chunk += BUFS) {
    if (!one(chunk, std::integral_constant<int, 0>{})) break;
    if (!one(chunk + 1, std::integral_constant<int, 1>{})) break;
    if constexpr (BUFS == 3) {
      if (!one(chunk + 2, std::integral_constant<int, 2>{})) break;
    }
  }

  const float part = L[0] + L[1], l = part + other_half(part), inv = 1.f / l;
  unsigned r[2][8];
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int e = 0; e < 16; e += 2)
      r[dt][e / 2] = __builtin_bit_cast(unsigned, bf16x2{(__bf16)(O[dt][e] * inv), (__bf16)(O[dt][e + 1] * inv)});
  const bool shared = is_shared(un.k);
  if (unit < 0 || (shared && partner)) return;           // (the conditional workgroup writes this row)
  if (row_ok) {
    __bf16* op = (__bf16*)a.o + b * a.os[0] + h * a.os[1] + checked_index(a.hdr, row, a.q_len) * a.os[2] + 8 * hh;
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        // dims 32 dt + 16 j .. + 15 of the query: its lanes hold 4 of each 8; exchanged, 8 in a row
        const auto x0 = __builtin_amdgcn_permlane32_swap(r[dt][4 * j], r[dt][4 * j + 2], false, false);
        const auto x1 = __builtin_amdgcn_permlane32_swap(r[dt][4 * j + 1], r[dt][4 * j + 3], false, false);
        const u32x4 piece = {x0[0], x1[0], x0[1], x1[1]};
        *(u32x4*)(op + 32 * dt + 16 * j) = piece;
        if (shared) *(u32x4*)(op + (a.B / 2) * a.os[0] + 32 * dt + 16 * j) = piece;
      }
  }
  // Rows whose reference went too far, and rows whose products with V may have overflowed although V and the result are
  // in range -- not finite, and formed under sums that a reference which follows each score would not have let grow --
  // are formed once more, the latter in the dimensions that are not finite.
  far &= queries;
  moved = (moved | __builtin_amdgcn_ballot_w64(l > 64.f * (float)wave_keys)) & queries;
  if (__builtin_expect((far | moved) != 0, 0)) {
    float any = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) any = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, r[e >> 3][e & 7]), kOnes, any, false);
    const uint64_t bad = (__builtin_amdgcn_ballot_w64(not_finite(any)) & moved) | far;
    if (bad != 0)
      attend_rows<false>(a, c, b, h, shared, (unsigned)(bad | (bad >> 32)), row,
                         __builtin_amdgcn_inverse_ballot_w64(far) ? ~0u : not_finite_dims(r),
                         [&](int) { return AllKeys{wave_keys, (wave_keys + 31) / 32}; });
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
  // Eight waves per workgroup halve the passes over K and V, four leave less of a workgroup idle and more of the chip
  // at work.  Up to four units: four waves.  Up to eight units, (B H, rows, keys), four / eight waves: where eight take
  // the place of a second workgroup of four on the CU (256, 169, 680: 13.0 / 12.2 us; 256, 256, 680: 21.3 / 19.7) and, over
  // many keys, where four would not be resident at once (480, 256, 680: 33.6 / 31.6; 480, 144, 1744: 58.5 / 50.1; but 600, 144,
  // 174: 15.5 / 16.4; 300, 256, 680: 26.7 / 28.0).  More units: where the last workgroup of a pair is nearly full and there are many
  // (288, 2240 tokens: 293 / 271; 60, 1024, 2240: 46.3 / 43.6; 480, 680, 680: 60.2 / 58.0; but 120, 680, 680: 17.6 / 19.2; 480, 243, 243:
  // 17.0 / 18.9; 2, 34 240: 476 / 590).
  // Two buffers instead of three let a fourth workgroup of four waves onto the CU, for a second barrier: from 512
  // workgroups on (900 workgroups, 216 rows: 13.6 / 12.0; 600, 100 rows: 14.6 / 14.3; but 120, 256 rows: 13.2 / 14.0).
  const int64_t BH = (int64_t)a.B * a.H, fours = BH * ((d.n_units + 3) / 4), eights = BH * ((d.n_units + 7) / 8);
  const int keys = d.off[d.qe];
  bool eight = false;
  if (d.n_units > 8)
    eight = BH * a.q_len >= 300 * 256 && 10 * (int64_t)BH * d.n_units >= 8 * 8 * eights && (eights >= 1024 || keys >= 1024);
  else if (d.n_units > 4)
    eight = (fours > 256 && fours <= 512) || (fours > 768 && keys >= 512);
  const int nwv = eight ? 8 : 4;
  const int64_t blocks = BH * ((d.n_units + nwv - 1) / nwv);
  if (blocks > 0x7fffffff) return fail(LITEVAR_E_UNSUPPORTED, "grid too large");
  d.bh_magic = (uint32_t)(((uint64_t)1 << 32) / (uint64_t)BH - (BH <= 1));
  const float c = a.sm_scale * 1.4426950408889634f;
  return launch_in_parts(blocks, nwv * 64, "dense bf16 attention launch", [&](int64_t first, unsigned n) {
    d.a.first_block = (uint32_t)first;
    if (nwv == 8) hipLaunchKernelGGL((k_attn_bf16_dense<8, 3>), dim3(n), dim3(nwv * 64), 0, st, d, c);
    else if (blocks > 512) hipLaunchKernelGGL((k_attn_bf16_dense<4, 2>), dim3(n), dim3(nwv * 64), 0, st, d, c);
    else hipLaunchKernelGGL((k_attn_bf16_dense<4, 3>), dim3(n), dim3(nwv * 64), 0, st, d, c);
  });
}

}  // namespace lv
