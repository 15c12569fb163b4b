// Device helpers shared by the bf16 attention kernels (gfx950): vector typedefs, the
// transposing LDS read, lane-mask select, the cross-row maximum and the LDS / vmcnt
// primitives that must not wait for outstanding LDS-DMA loads.
#pragma once
#include "internal.h"

namespace lv {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((address_space(3))) void lds_void;
typedef const __attribute__((address_space(1))) void global_void;
// constant address space: a load from a wave-uniform address becomes a scalar load
typedef const __attribute__((address_space(4))) uint64_t* const_u64_ptr;
typedef const __attribute__((address_space(4))) int32_t* const_i32_ptr;

constexpr float kFloor = -1.0e30f;   // initial softmax reference: keeps exp2 arguments finite
constexpr float kSlack = 6.0f;       // base-2 exponent by which a score may exceed the reference
// Row sums outside move the reference of the windowed 32-query kernel.  From 2^-10 on, products with the smallest normal V
// keep 13 bits above fp32's smallest subnormal; above 2^40 they may overflow, which ends in attend_row.  (A move leaves a sum
// of at least 2^-0.5.  At 1 as the lower end, rows of one large probability moved in every step: 2240 tokens, 288 pairs,
// scores of mean -24 and standard deviation 6 159 -> 218 us; 164 with a reference that moves once.)
constexpr float kMostSum = 0x1p40f, kLeastSum = 0x1p-10f;

__device__ inline bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

__device__ inline s16x4 lds_read_tr16(const unsigned char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p));
}

// keep `s` where the lane's bit of the wave-uniform `mask` is set, else -inf
// (inverse ballot: the SGPR pair becomes the select condition of one v_cndmask)
__device__ inline float mask_select(float s, uint64_t mask) {
  return __builtin_amdgcn_inverse_ballot_w64(mask) ? s : -INFINITY;
}

// max over the four lanes l, l^16, l^32, l^48: v_permlane32_swap exchanges the upper half
// of its first register with the lower half of its second, v_permlane16_swap the odd
// 16-lane rows of the first with the even rows of the second.  (The two results are
// copied into scalars before the float reinterpretation: a __builtin_bit_cast applied
// directly to an element of the returned vector reads element 0 for both.)
__device__ inline float max_across_rows(float x) {
  const unsigned u = __float_as_uint(x);
  auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const unsigned a0 = a[0], a1 = a[1];
  const unsigned v = __float_as_uint(fmaxf(__uint_as_float(a0), __uint_as_float(a1)));
  auto b = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  const unsigned b0 = b[0], b1 = b[1];
  return fmaxf(__uint_as_float(b0), __uint_as_float(b1));
}

constexpr bf16x2 kOnes = {(__bf16)1.0f, (__bf16)1.0f};

// the value in the other lane of a query (l ^ 32)
__device__ inline float other_half(float x) {
  const unsigned u = __float_as_uint(x);
  auto sw = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const unsigned s0 = sw[0], s1 = sw[1];       // (lower half's value, upper half's value) in every lane
  return __uint_as_float((threadIdx.x & 32) ? s0 : s1);
}

// (on the bits, behind a barrier for the optimiser: the build lets it assume that no value is NaN)
__device__ inline bool not_finite(float x) {
  unsigned u = __float_as_uint(x);
  asm volatile("" : "+v"(u));
  return (u & 0x7f800000u) == 0x7f800000u;
}

__device__ inline unsigned lds_addr(const void* p) {
  return (unsigned)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}

// waits for LDS reads that inline assembly has issued; the operands are tied so that no use is scheduled above
__device__ inline void lds_wait_k(u32x4& k00, u32x4& k01, u32x4& k10, u32x4& k11) {
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(k00), "+v"(k01), "+v"(k10), "+v"(k11) : : "memory");
}

__device__ inline void lds_wait_v_wide(u32x2 (&va)[8]) {
  asm volatile("s_waitcnt lgkmcnt(0)"
               : "+v"(va[0]), "+v"(va[1]), "+v"(va[2]), "+v"(va[3]), "+v"(va[4]), "+v"(va[5]), "+v"(va[6]),
                 "+v"(va[7]) : : "memory");
}

// What every attention kernel checks before it reads anything else of the plan: the blob's
// header carries the magic and not the builder's error mark.  A zeroed, stale or half-built
// blob then makes the launch a no-op instead of a walk over garbage.  (Scalar loads: the
// header is the same for every workgroup.)
__device__ inline bool plan_usable(const Header* hdr) {
  const const_i32_ptr w = (const_i32_ptr)hdr;
  int magic_lo = w[0], magic_hi = w[1], err = w[offsetof(Header, error) / 4];
  asm volatile("" : "+s"(magic_lo), "+s"(magic_hi), "+s"(err));   // one round trip for the three words
  return magic_lo == (int32_t)(kMagic & 0xffffffffu) && magic_hi == (int32_t)(kMagic >> 32) && err != kErrBuilder;
}

// The bounds-checking build (-DLITEVAR_DEBUG_BOUNDS, a second library for tests and for chasing
// a suspected plan/kernel mismatch): every token that addresses a K/V row, every query row
// that addresses Q or O (from the plan, or from the dense kernel's own units and tiles) and every LDS
// offset taken from a step descriptor is compared with its limit before use; a value out of range is replaced by 0 and the plan's header is
// marked (litevar_plan_check then says so).  The normal build compiles the checks away.
__device__ inline int checked_index([[maybe_unused]] Header* hdr, int value, [[maybe_unused]] int limit) {
#ifdef LITEVAR_DEBUG_BOUNDS
  if ((unsigned)value >= (unsigned)limit) { hdr->error = kErrBounds; return 0; }
#endif
  return value;
}

// A softmax reference that is subtracted from scaled scores is a multiple of its own rounding, so that the largest
// probability is off by up to 2^(2^-25 m): nothing below 2^24, everything from 2^31 on.  Queries whose reference
// gets there are formed again by attend_row, which subtracts the largest score before it scales.
constexpr float kFarReference = 0x1p24f;
__device__ inline uint64_t is_far(float negm) { return __builtin_amdgcn_ballot_w64(!(fabsf(negm) < kFarReference)); }

template <int N> __device__ inline void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
  // gfx9 encoding: vmcnt[3:0] in bits 3:0, vmcnt[5:4] in bits 15:14; expcnt/lgkmcnt left at max
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0f70);
}

// (counted anew, where threadIdx.x would hold a register from the kernel's start)
__device__ inline int lane_of_wave() { return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }

// One query row of pair (b, h), by all 64 lanes of a wave, for results that the matrix products cannot give: 32 keys at a
// time, lane i and lane i + 32 the two halves of key i's score, then lane d head dimension d of the output.  Nothing
// is formed from a key that the query does not keep, and the softmax reference is the largest score itself, so that
// any scores that fp32 holds give their probabilities.  mine: the lane's dimension is stored; once none of these is finite
// any more, the rest of the keys is left.
// keys.key(block, i, tok): the query keeps key i of block `block`, which is token `tok`; keys.n_blocks blocks.
// Bound: about 400 instructions and two trips to memory for 32 keys.  2240 tokens, 288 pairs, a bad V element in a token
// that all queries keep, K all NaN, a bad V element in a late token: 1.3 / 0.9 / 3.2 ms a call (with a row per lane, key
// by key and to the end: 10.8 / 12.9 / 2.9).
template <bool Q8, class Keys>
__device__ inline void attend_row(const AttnArgs& a, float c, int b, int h, int qrow, bool shared, bool mine,
                                  const Keys keys) {
  constexpr int kElem = Q8 ? 1 : 2;
  const int lane = lane_of_wave(), i = lane & 31, first_dim = lane & 32;
  const int64_t kv_at = (b * a.ks[0] + h * a.ks[1]) * kElem, pair = (int64_t)b * a.H + h;
  const unsigned char *K = (const unsigned char*)a.k + kv_at, *V = (const unsigned char*)a.v + kv_at;
  const unsigned row_bytes = (unsigned)a.ks[2] * kElem;    // (a (batch, head) slab spans < 2 GiB)
  [[maybe_unused]] const int64_t first_row = Q8 ? pair * (a.ks[1] / a.ks[2]) : 0;
  qrow = checked_index(a.hdr, qrow, a.q_len);
  // 32 dimensions of a row: bf16, or 8-bit codes with the row's (scale, zero point) as the kernels convert them
  auto load_half = [&](const unsigned char* row, [[maybe_unused]] const float2* sz, float (&x)[32]) {
    const u32x4* p = (const u32x4*)(row + first_dim * kElem);
    u32x4 raw[2 * kElem];
#pragma unroll
    for (int t = 0; t < 2 * kElem; ++t) raw[t] = p[t];
    float2 f = make_float2(0.f, 0.f);
    if constexpr (Q8) f = *sz;
#pragma unroll
    for (int e = 0; e < 32; ++e) {
      if constexpr (Q8) x[e] = (float)(__bf16)fmaf(f.x, (float)(int8_t)((raw[e >> 4][(e >> 2) & 3] >> (8 * (e & 3))) & 0xffu), f.y);
      else x[e] = __uint_as_float(e & 1 ? raw[e >> 3][(e >> 1) & 3] & 0xffff0000u : raw[e >> 3][(e >> 1) & 3] << 16);
    }
  };
  float q[32];
  load_half((const unsigned char*)a.q + (b * a.qs[0] + h * a.qs[1] + qrow * a.qs[2]) * kElem,
            Q8 ? a.q_sz + pair * a.q_len + qrow : nullptr, q);
  float m = -INFINITY, l = 0.f, o = 0.f;
  bool nan = false;                            // a kept key's score is
  for (int block = 0; block < keys.n_blocks; ++block) {
    int tok = 0;
    const bool keep = keys.key(block, i, tok);
    const unsigned kept = (unsigned)__builtin_amdgcn_ballot_w64(keep);
    if (kept == 0) continue;
    tok = checked_index(a.hdr, keep ? tok : __builtin_amdgcn_readlane(tok, __builtin_ctz(kept)), a.kv_len);
    float dot = 0.f, x[32];
    load_half(K + (unsigned)tok * row_bytes, Q8 ? a.k_sz + first_row + tok : nullptr, x);
#pragma unroll
    for (int e = 0; e < 32; ++e) dot = fmaf(q[e], x[e], dot);
    dot += __shfl_xor(dot, 32);
    unsigned bits = __float_as_uint(dot);
    asm volatile("" : "+v"(bits));             // (see not_finite)
    if ((nan = __builtin_amdgcn_ballot_w64(keep && (bits & 0x7fffffffu) > 0x7f800000u) != 0)) break;
    float mx = keep ? dot : -INFINITY;
#pragma unroll
    for (int d = 16; d > 0; d >>= 1) mx = fmaxf(mx, __shfl_xor(mx, d));
    const float m_new = fmaxf(m, mx);
    const float p = keep ? __builtin_amdgcn_exp2f((dot - m_new) * c) : 0.f;
    const float alpha = m > -INFINITY ? __builtin_amdgcn_exp2f((m - m_new) * c) : 0.f;
    float sum = p;
#pragma unroll
    for (int d = 16; d > 0; d >>= 1) sum += __shfl_xor(sum, d);
    if (m_new == -INFINITY) continue;          // (only scores of -inf so far)
    l = fmaf(l, alpha, sum); m = m_new; o *= alpha;
#pragma unroll
    for (int j0 = 0; j0 < 32; j0 += 16) {      // (sixteen rows of V in flight)
      float v[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int t = __builtin_amdgcn_readlane(tok, j0 + j);
        const unsigned char* row = V + (unsigned)t * row_bytes;      // (in scalar registers)
        if constexpr (Q8) {
          const float2 f = a.v_sz[first_row + t];
          v[j] = (float)(__bf16)fmaf(f.x, (float)((const int8_t*)row)[lane], f.y);
        } else {
          v[j] = (float)((const __bf16*)row)[lane];
        }
      }
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const float pj = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(p), j0 + j));
        o = (kept >> (j0 + j)) & 1u ? fmaf(pj, v[j], o) : o;
      }
    }
    if (not_finite(l) || __builtin_amdgcn_ballot_w64(mine && !not_finite(o)) == 0) break;
  }
  if (!mine) return;
  __bf16* op = (__bf16*)a.o + b * a.os[0] + h * a.os[1] + qrow * a.os[2] + lane;
  const __bf16 r = nan ? __builtin_bit_cast(__bf16, (unsigned short)0x7fc0) : (__bf16)(o * (1.f / l));
  *op = r;
  if (shared) op[(a.B / 2) * a.os[0]] = r;
}

// Which of a query's 32 values in this lane (r: pairs of bf16, dims 32 dt + 8 j + 4 (lane / 32) .. + 3 of a 32 x 32 tile's
// column, in that order) are not finite.
__device__ inline unsigned not_finite_dims(const unsigned (&r)[2][8]) {
  unsigned bits = 0;
#pragma unroll
  for (int e = 0; e < 32; ++e)
    bits |= (unsigned)(((r[e >> 4][(e & 15) >> 1] >> (16 * (e & 1))) & 0x7f80u) == 0x7f80u) << e;
  return bits;
}

// attend_row for the rows of the lanes in `rows` (their row: `row`), behind the store of the wave's results: the
// dimensions dims of a lane and of the one 32 above it are stored again.
template <bool Q8, class KeysOf>
__device__ inline void attend_rows(const AttnArgs& a, float c, int b, int h, bool shared, unsigned rows, int row, unsigned dims, KeysOf keys_of) {
  for (; __builtin_expect(rows != 0, 0); rows &= rows - 1) {
    wait_vmcnt<0>();                           // (what is stored next goes to places that were just stored to)
    const int at = __builtin_ctz(rows), r = __builtin_amdgcn_readlane(row, at), l = lane_of_wave();
    // lane d for dimension d: value 16 (d / 32) + 4 (d / 8 % 4) + d % 4 of the query's lane half d / 4 % 2
    const unsigned lo = __builtin_amdgcn_readlane(dims, at), up = __builtin_amdgcn_readlane(dims, at + 32);
    const bool mine = ((l & 4 ? up : lo) >> (16 * (l >> 5) + 4 * ((l >> 3) & 3) + (l & 3))) & 1u;
    attend_row<Q8>(a, c, b, h, r, shared, mine, keys_of(r));
  }
}

// x = q n + r for a divisor n whose magic = floor(2^32 / n) came with the kernel arguments
// (n = 1: magic = 2^32 - 1): the estimate floor(x magic / 2^32) is the quotient or one below it
// for every x < 2^32, so one correction step makes it exact.
__device__ inline void divmod_by(uint32_t x, uint32_t n, uint32_t magic, int& q, int& r) {
  uint32_t qq = __umulhi(x, magic), rr = x - qq * n;
  if (rr >= n) { ++qq; rr -= n; }
  q = (int)qq; r = (int)rr;
}

// The work item of this workgroup (the host's spread_over_xcds): item `item` of pair bh, which is the
// me-th pair of its XCDs.  false: none.
__device__ inline bool xcd_item(const AttnArgs& a, int items, int& me, int& bh, int& item) {
  uint32_t block = a.first_block;
  asm volatile("" : "+s"(block), "+s"(items));   // one scalar round trip for both (left alone, items' load waits: 0.6 % of a call)
  block += blockIdx.x;
  const int xcd = block & 7;
  int in_part;
  divmod_by(block >> 3, (uint32_t)a.part, a.part_magic, me, in_part);
  bh = me * (8 >> a.spread_log) + (xcd >> a.spread_log);
  item = (in_part << a.spread_log) + (xcd & ((1 << a.spread_log) - 1));
  return bh < a.B * a.H && item < items;
}

// N consecutive-stride LDS words (stride 32 bytes) written by earlier LDS-DMA loads of this
// wave whose completion the caller has already established.  Inline assembly, because the
// compiler would otherwise order these reads after a vmcnt(0) wait (it cannot know which
// DMA loads have landed) and so drain the prefetch queue.
template <int N> __device__ inline void lds_read_tokens(const int32_t* p, int (&t)[N]);
template <> __device__ inline void lds_read_tokens<4>(const int32_t* p, int (&t)[4]) {
  const unsigned a = (unsigned)(uintptr_t)(__attribute__((address_space(3))) const int32_t*)p;
  asm volatile("ds_read_b32 %0, %4\n\tds_read_b32 %1, %4 offset:32\n\t"
               "ds_read_b32 %2, %4 offset:64\n\tds_read_b32 %3, %4 offset:96\n\t"
               "s_waitcnt lgkmcnt(0)"
               : "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3]) : "v"(a) : "memory");
}
template <> __device__ inline void lds_read_tokens<8>(const int32_t* p, int (&t)[8]) {
  const unsigned a = (unsigned)(uintptr_t)(__attribute__((address_space(3))) const int32_t*)p;
  asm volatile("ds_read_b32 %0, %8\n\tds_read_b32 %1, %8 offset:32\n\t"
               "ds_read_b32 %2, %8 offset:64\n\tds_read_b32 %3, %8 offset:96\n\t"
               "ds_read_b32 %4, %8 offset:128\n\tds_read_b32 %5, %8 offset:160\n\t"
               "ds_read_b32 %6, %8 offset:192\n\tds_read_b32 %7, %8 offset:224\n\t"
               "s_waitcnt lgkmcnt(0)"
               : "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3]), "=&v"(t[4]), "=&v"(t[5]),
                 "=&v"(t[6]), "=&v"(t[7]) : "v"(a) : "memory");
}

// LDS accesses of the loader wave that must not wait for its outstanding LDS-DMA loads
// (the compiler orders ordinary LDS accesses after vmcnt(0) once a DMA load is pending)
__device__ inline void lds_store_i32_nowait(int32_t* p, int v) {
  const unsigned a = (unsigned)(uintptr_t)(__attribute__((address_space(3))) int32_t*)p;
  asm volatile("ds_write_b32 %0, %1" : : "v"(a), "v"(v) : "memory");
}
__device__ inline int lds_load_i32_nowait(const int32_t* p) {   // waits for LDS only, not for vector memory
  const unsigned a = (unsigned)(uintptr_t)(__attribute__((address_space(3))) const int32_t*)p;
  int v;
  asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(a) : "memory");
  return v;
}
template <int NW> __device__ inline int lds_min_progress(const int32_t* p) {
  static_assert(NW == 4 || NW == 8, "progress words are read four at a time");
  const unsigned a = (unsigned)(uintptr_t)(__attribute__((address_space(3))) const int32_t*)p;
  typedef __attribute__((ext_vector_type(4))) int i32x4;
  i32x4 x, y;
  if constexpr (NW == 8) {
    asm volatile("ds_read_b128 %0, %2\n\tds_read_b128 %1, %2 offset:16\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(x), "=&v"(y) : "v"(a) : "memory");
  } else {
    asm volatile("ds_read_b128 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(x) : "v"(a) : "memory");
    y = x;
  }
  const int m0 = min(min(x[0], x[1]), min(x[2], x[3])), m1 = min(min(y[0], y[1]), min(y[2], y[3]));
  return min(m0, m1);
}

}  // namespace lv
