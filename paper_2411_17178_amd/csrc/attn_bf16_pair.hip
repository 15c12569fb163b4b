// bf16 windowed attention forward for gfx950 (CDNA4), Section 2 of the paper, for plans
// with 16 patches per group: O = softmax(sm_scale * Q K^T over the kept keys) V, with the
// Section 3 cond -> uncond output reuse folded into the store.
//
// One workgroup = eight waves = one group of up to 16 x 16 queries of one scale of one (batch, head), which its
// wide patches tile: every wave owns 32 queries (4 x 8, or whatever covers the group best) and one eighth of the
// loading.  (A second form, sixteen waves with a patch of 16 queries each, serves plans without wide patches.)
//
// Why 32 queries per wave: what bounds a step is the vector issue of its SIMD, four waves of which run steps at the same
// time, and its own chain of latencies.  A step of 32 keys costs 69 vector and 9 matrix instructions for 32 queries
// (v_mfma_f32_32x32x16_bf16), where 16 queries (v_mfma_f32_16x16x32_bf16) took 45 and 9, for 1.13 to 1.18 times the pairs.
// The descriptor carries the step's mask, so that nothing on the step's way waits for a scalar load.
// Measured against two 16-query patches per wave: 2240 tokens, radius 4, 288 pairs 176.5 -> 159.7 us; 34 240 tokens, 32 pairs
// with sharing 393 -> 321 us; 256 queries on 680 keys, 480 pairs 29.3 -> 28.6 us, 240 working pairs of ten steps 90.9 -> 87.7
// us (there against one 16-query patch per wave).  Of a wave's time at 2240 tokens (31 000 cycles): start-up 22 % (the loads
// before the first barrier pass the CU's address unit at 64 bytes a cycle, then a trip to memory), steps 40 %, barriers
// 20 %, waits for loads 10 %.
//
// The group's key list is streamed once through an LDS ring of five chunks of 64 keys
// (one 128-byte K row and one 128-byte V row per key, 16-byte pieces XOR-swizzled by
// slot; 80 KiB, so that two workgroups share a CU); chunk t lives in slot t mod 5.  The
// plan counts NC chunks; the kernel runs P = NC / 2 + 1 phases: phase 0 is chunk 0 alone
// (the first steps start on as little data as possible), phase p >= 1 is chunks 2p-1 and
// 2p, i.e. the steps whose last key lies in one of them.  A step spans at most two
// consecutive chunks, so a step that ends in chunk t reads chunks t-1 .. t: phase p reads
// chunks 2p-2 .. 2p, which are three of the five slots; the other two slots held chunks
// 2p-4 and 2p-3, which nobody reads after the barrier that ended phase p-1, and receive
// chunks 2p+1 and 2p+2 (phase p+1) while phase p computes.
//   Prologue: all scalar plan words, then the tokens of the first chunks, the first step descriptors, Q and the other
//     small loads, then chunks 0, 1 and 2 (which wait for the tokens only where the list does not start with whole key
//     scales).  With at most chunks 1 and 2 outstanding (a wave issues PW transfers per chunk: vmcnt 2 PW) comes the
//     first barrier: Q, the descriptors and chunk 0 are in.
//   Phase p: a wave
//     issues the descriptor loads of its steps of this phase beyond the first,
//     runs the first step,
//     waits for all its vector memory operations (p >= 1: the descriptors just requested;
//       chunks 2p-1 and 2p were waited for at the end of phase p-1),
//     requests the first descriptor and the tokens of phase p+1 and then issues its share
//       of chunks 2p+1 and 2p+2 (p >= 1; in phase 0 chunks 1 and 2 are already in flight) --
//       not right behind the barrier, where the loads of all eight waves would queue up in
//       front of the first K reads, and behind the small loads, because a load issued behind
//       a chunk is held up until the chunk's data is in,
//     runs its other steps, waits for all its vector memory operations (vmcnt 0: the chunks
//       of phase p+1 have landed) and joins the barrier.
// Two chunks (32 KiB) per workgroup are in flight during a phase, and a key row is moved
// from HBM/L2 to LDS exactly once per (batch, head, group).
//
// A wave that issues LDS-DMA loads must read LDS through inline assembly: the compiler
// cannot tell which of them a plain LDS read depends on and would wait for all
// (vmcnt(0)) before every read.  And no loaded register may be copied or loaded again under a condition while transfers
// are in flight: the compiler then waits for everything at the copy (tokens that were loaded only where the list needs
// them cost 5 % of a launch that way).
//
// Step arithmetic (16 queries) is that of the 8-patch kernel: S^T = K_tile . Q^T by
// v_mfma_f32_16x16x32_bf16 (a lane owns one query column and four keys per tile) on
// accumulators that start at minus the softmax reference where the scalar lane mask keeps the
// pair and at -inf elsewhere (one v_cndmask per score), so the tiles leave the matrix pipe as
// masked scores relative to the reference; base-2 online softmax with a lazily updated
// reference, O^T += V^T . P^T with ds_read_b64_tr_b16 operands, row sums by a fifth MFMA.
// (Folding the softmax scale into Q, which would save the multiplication per score, costs a
// second bf16 rounding of Q: with peaked attention -- scores of some tens -- the output
// error grows tenfold.  The scale is applied in fp32.)
#include <type_traits>

#include "attn_bf16_common.h"

namespace lv {

namespace {

constexpr int kGroupPatches = 16;     // query patches per workgroup
constexpr int kDmaKeys = 64;          // keys per chunk (the unit of loading and of ring slot reuse)
constexpr int kRingChunks = 5;        // ring depth: look-back, two current, two landing
constexpr int kBufferFlags = 0x00020000;   // word 3 of a raw buffer resource on gfx9: 32-bit data format
typedef __attribute__((ext_vector_type(2))) short s16x2;
constexpr int kBoostPhases = 3;       // phases that a later-arrived workgroup runs at raised priority
constexpr float kMaskB = 2.0f;        // of the mask product (see run_step32): times -2^127 it is -inf
constexpr int kLater = 2;             // descriptors, beyond the first step of a phase, that are fetched at
                                      // the start of the phase

// four 16-byte K pieces (two keys x two halves of the head dimension): issued only,
// lds_wait_k() must precede the first use
__device__ inline void lds_read_k_issue(unsigned a0, unsigned a1, u32x4& k00, u32x4& k01, u32x4& k10, u32x4& k11) {
  asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\t"
               "ds_read_b128 %2, %6\n\tds_read_b128 %3, %7"
               : "=&v"(k00), "=&v"(k01), "=&v"(k10), "=&v"(k11)
               : "v"(a0), "v"(a0 ^ 16u), "v"(a1), "v"(a1 ^ 16u) : "memory");
}

// transposing reads of the V^T operands of one step (4 head-dim tiles x 2 key halves);
// issued only: lds_wait() must precede the first use
template <int VOFF>
__device__ inline void lds_read_v(unsigned v0, unsigned v1, const unsigned (&x)[3][2], uint2 (&va)[4][2]) {
  asm volatile("ds_read_b64_tr_b16 %0, %8 offset:%16\n\tds_read_b64_tr_b16 %1, %9 offset:%16\n\t"
               "ds_read_b64_tr_b16 %2, %10 offset:%16\n\tds_read_b64_tr_b16 %3, %11 offset:%16\n\t"
               "ds_read_b64_tr_b16 %4, %12 offset:%16\n\tds_read_b64_tr_b16 %5, %13 offset:%16\n\t"
               "ds_read_b64_tr_b16 %6, %14 offset:%16\n\tds_read_b64_tr_b16 %7, %15 offset:%16"
               : "=&v"(va[0][0]), "=&v"(va[0][1]), "=&v"(va[1][0]), "=&v"(va[1][1]),
                 "=&v"(va[2][0]), "=&v"(va[2][1]), "=&v"(va[3][0]), "=&v"(va[3][1])
               : "v"(v0), "v"(v1), "v"(x[0][0]), "v"(x[0][1]), "v"(x[1][0]), "v"(x[1][1]),
                 "v"(x[2][0]), "v"(x[2][1]), "i"(VOFF) : "memory");
}

// waits for the reads issued by lds_read_v; the operands are tied so that no use is
// scheduled above the wait
__device__ inline void lds_wait(uint2 (&va)[4][2]) {
  asm volatile("s_waitcnt lgkmcnt(0)"
               : "+v"(va[0][0]), "+v"(va[0][1]), "+v"(va[1][0]), "+v"(va[1][1]),
                 "+v"(va[2][0]), "+v"(va[2][1]), "+v"(va[3][0]), "+v"(va[3][1]) : : "memory");
}

// the same for a wide patch: four 16-byte pieces of one key's K row ...
__device__ inline void lds_read_k_row_issue(unsigned k, u32x4 (&r)[4]) {
  asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\t"
               "ds_read_b128 %2, %6\n\tds_read_b128 %3, %7"
               : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3])
               : "v"(k), "v"(k ^ 32u), "v"(k ^ 64u), "v"(k ^ 96u) : "memory");
}
// ... and V^T: two slices of 16 keys (t), two halves of one (j), two head-dim tiles (dt); va[4 t + 2 j + dt]
template <int VOFF>
__device__ inline void lds_read_v_wide(const unsigned (&v)[4], const unsigned (&x)[4], u32x2 (&va)[8]) {
  asm volatile("ds_read_b64_tr_b16 %0, %8 offset:%16\n\tds_read_b64_tr_b16 %1, %9 offset:%16\n\t"
               "ds_read_b64_tr_b16 %2, %10 offset:%16\n\tds_read_b64_tr_b16 %3, %11 offset:%16\n\t"
               "ds_read_b64_tr_b16 %4, %12 offset:%16\n\tds_read_b64_tr_b16 %5, %13 offset:%16\n\t"
               "ds_read_b64_tr_b16 %6, %14 offset:%16\n\tds_read_b64_tr_b16 %7, %15 offset:%16"
               : "=&v"(va[0]), "=&v"(va[1]), "=&v"(va[2]), "=&v"(va[3]),
                 "=&v"(va[4]), "=&v"(va[5]), "=&v"(va[6]), "=&v"(va[7])
               : "v"(v[0]), "v"(x[0]), "v"(v[1]), "v"(x[1]), "v"(v[2]), "v"(x[2]), "v"(v[3]), "v"(x[3]),
                 "i"(VOFF) : "memory");
}
struct WideArgs {
  const WaveDesc* waves;  // the wide patches
  int boost;              // all workgroups of the launch are resident at once
};

struct WidePatchState {   // a wave's 32 queries
  bf16x8 q[4];            // Q^T as the B operand: lane (n, h) holds Q[query n][16 t + 8 h .. + 7]
  f32x16 O[2];            // O^T accumulators: dims 32 dt + 8 (e / 4) + 4 h + e % 4 of query n
  float L, negm;          // this lane's part of the row sum, minus the softmax reference m (base 2, whole numbers)
  uint64_t unset;         // lanes whose query's sum is still below kLeastSum
  uint64_t far;           // lanes whose reference was beyond kFarReference at some time
  bf16x8 b;               // B operand of the mask product, see run_step32
};

struct PatchState {       // one query patch of a wave
  bf16x8 qb0, qb1;        // Q^T as the B operand: lane (n, g4) holds Q[query n][16 g4 .. +15]
  f32x4 O[4], Lacc;       // O^T accumulators and row sums
  float thr, negm;        // minus the softmax reference m; thr = how far a score may rise above m
                          // before m moves: kFloor while m is unset
};

// The keys of one query for attend_row, in the steps of the patch of 16 that holds the query's row, one of the group's
// sixteen from `patches` on
struct StepKeys {
  const AttnArgs& a;
  int64_t step0; int n_blocks, column;
  __device__ StepKeys(const AttnArgs& args, const WaveDesc* patches, int qrow) : a(args), step0(0), n_blocks(0), column(0) {
    const WaveDesc wd = patches[lane_of_wave() & (kGroupPatches - 1)];
    const int d = qrow - wd.q_base, dy = d / max((int)wd.sk, 1), dx = d - dy * wd.sk;
    const bool holds = d >= 0 && dy < kPatch && dx < kPatch && ((wd.valid >> (kPatch * dy + dx)) & 1u);
    const uint64_t who = __builtin_amdgcn_ballot_w64(holds);
    if (who == 0) return;
    const int at = __builtin_ctzll(who);
    step0 = __builtin_amdgcn_readlane(wd.step_begin, at);
    n_blocks = __builtin_amdgcn_readlane(wd.n_steps, at);
    column = __builtin_amdgcn_readlane(kPatch * dy + dx, at);
  }
  __device__ bool key(int block, int i, int& tok) const {
    const int64_t s = step0 + block;
    const int r = i & 15;
    tok = a.step_tok[s * kStepKeys + i];
    return (a.step_mask[s * 8 + 4 * (i >> 4) + (r & 3)] >> ((r >> 2) * 16 + column)) & 1;
  }
};

}  // namespace

// PW = 2: a wide patch, 32 queries, per wave (8 waves per workgroup, two workgroups per CU); PW = 1: a patch of 16
// queries per wave (16 waves per workgroup, one workgroup per CU).  A plan is laid out for one of them: the
// steps and the order of the key list are that form's; with 16 waves the loading duty of a chunk is one K or one V transfer
// per wave.
//
// Q8 (Section 4, 8-bit Q, K, V): the operands are int8 codes with one (scale, zero point) per
// token row.  A wave's share of a chunk then comes through registers instead of LDS-DMA: one
// 16-byte load of codes and one of the row's parameters per lane (lanes 0-31 K rows, lanes
// 32-63 V rows with eight waves; K waves and V waves with sixteen), requested where the bf16
// form issues its transfers, converted to bf16(s code + z) and written to the ring -- same
// slots, same swizzle -- at the end of the phase, before the barrier.  Steps, masks and
// epilogue are the same code; the ring holds exactly what a dequantised bf16 copy would put
// there, so the results equal those of the bf16 kernel on such a copy bit for bit.
template <int PW, bool Q8>
__global__ __launch_bounds__((kGroupPatches / PW) * 64) __attribute__((amdgpu_waves_per_eu(4, 4)))
void k_attn_bf16_pair(AttnArgs a, WideArgs wide, float c) {
  constexpr bool WIDE = PW == 2;                   // the group's wide patches (32 queries), else its patches (16)
  constexpr int C = kDmaKeys;
  constexpr int R = kRingChunks * C;               // ring slots
  constexpr int VOFF = R * kRingRowBytes;          // V ring follows the K ring
  __shared__ __align__(1024) unsigned char smem[2 * R * kRingRowBytes];
  unsigned char* const Kring = smem;
  unsigned char* const Vring = smem + VOFF;

  int me, grp, bh, b, h;                  // me: which of the (batch, head) pairs of this XCD
  if (!xcd_item(a, a.n_groups, me, bh, grp)) return;
  divmod_by((uint32_t)bh, (uint32_t)a.H, a.H_magic, b, h);
  // Scalar round trip 1: the header words that say whether the plan may be used at all (a
  // zeroed, stale or half-built blob makes the launch a no-op) and, for plans with a radius
  // table per head, the head's group, whose copy of the work-list this workgroup walks.
  // (Requested together and tied to one point, so that they cost one round trip, not four.)
  const const_i32_ptr hw = (const_i32_ptr)a.hdr;
  int magic_lo = hw[0], magic_hi = hw[1], herr = hw[offsetof(Header, error) / 4], hg = 0;
  if (a.head_map) hg = ((const_i32_ptr)a.head_map)[h];
  asm volatile("" : "+s"(magic_lo), "+s"(magic_hi), "+s"(herr), "+s"(hg));
  if (magic_lo != (int32_t)(kMagic & 0xffffffffu) || magic_hi != (int32_t)(kMagic >> 32) || herr == kErrBuilder) return;
  const int grp_g = grp + hg * a.n_groups;
  // Scalar round trip 2 (together with the patch descriptors below): the group descriptor.
  const const_i32_ptr gw = (const_i32_ptr)(a.groups + grp_g);
  GroupDesc gd;
  gd.union_base = gw[0]; gd.n_union = gw[1]; gd.n_phases = gw[2]; gd.k = gw[3];
  gd.gy = gw[4]; gd.gx = gw[5]; gd.phase_base = gw[6]; gd.ident = gw[7];

  // Two workgroups share a CU, and the instruction arbiter prefers the older waves: left
  // alone, the workgroup that arrived first runs as if it had the CU to itself and the other
  // one finishes a quarter later, alone on a CU that it cannot fill.  The later arrival (it
  // gets the higher wave slots of each SIMD) therefore runs at raised priority through its
  // first phases, which evens out the two finishing times (480 workgroups: 29.7 -> 28.5 us).  Only where the launch
  // is resident at once: with workgroups waiting for a place it is better to finish the older one (4608: 162.5, 159.7 without).
  const bool later_arrival = PW == 2 && wide.boost && (__builtin_amdgcn_s_getreg(4 | (3 << 11)) & 0xf) >= 2;   // HW_ID.WAVE_ID
  if (later_arrival) __builtin_amdgcn_s_setprio(1);
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int n = WIDE ? lane & 31 : lane & 15, hi = WIDE ? lane >> 5 : lane >> 4;   // query column, part of the other index
  // The plan counts 64-key chunks.  Phase 0 is chunk 0 alone, so that the first steps start
  // on the smallest possible amount of data; phase p >= 1 is chunks 2 p - 1 and 2 p.
  const int NC = __builtin_amdgcn_readfirstlane(gd.n_phases);   // chunks of the (padded) key list
  const int P = NC / 2 + 1;                                     // phases

  // ---- loading duty: rows [8 w, 8 w + 8) of every chunk, w = wave mod 8: K and V rows with
  // eight waves, K rows (waves 0-7) or V rows (waves 8-15) with sixteen ----
  constexpr int kElem = Q8 ? 1 : 2;                    // bytes per operand element
  const unsigned char* Kp = (const unsigned char*)a.k + (b * a.ks[0] + h * a.ks[1]) * kElem;
  const unsigned char* Vp = (const unsigned char*)a.v + (b * a.ks[0] + h * a.ks[1]) * kElem;
  const unsigned row_bytes = (unsigned)a.ks[2] * kElem;   // a (batch, head) slab spans < 2 GiB (checked by the API)
  const int32_t* utok = a.union_tok + gd.union_base;
  // bf16: eight lanes per 128-byte row; Q8: four lanes per 64-byte row of codes
  const int row = Q8 ? 8 * (wave & 7) + ((lane >> 2) & 7) : 8 * (wave & 7) + (lane >> 3);
  // A lane's row of chunk t goes to slot (t % 5) * 64 + row.  Chunks start at multiples of 64
  // slots, so the slot's swizzle -- and with it the 16-byte piece of the source row that
  // this lane fetches -- does not depend on t.
  const unsigned piece_off = (((unsigned)lane & 7u) ^ ring_swizzle((unsigned)row)) << 4;
  static_assert((kDmaKeys & 63) == 0, "the swizzle folds slot bits 0..5 only");
  auto row_at = [&](int tok) -> unsigned {             // this lane's piece of token tok's row
    return __umul24((unsigned)checked_index(a.hdr, tok, a.kv_len), row_bytes) + piece_off;   // (both below 2^24, checked by the API)
  };
  auto issue_chunk = [&](int t, unsigned src) {        // chunk t -> ring slots (t % 5) * 64 ...
    const int slot0 = (t % kRingChunks) * C + 8 * (wave & 7);
    if (PW == 2 || wave < 8)
      __builtin_amdgcn_global_load_lds((global_void*)(Kp + src), (lds_void*)(Kring + slot0 * kRingRowBytes), 16, 0, 0);
    if (PW == 2 || wave >= 8)
      __builtin_amdgcn_global_load_lds((global_void*)(Vp + src), (lds_void*)(Vring + slot0 * kRingRowBytes), 16, 0, 0);
  };
  constexpr int kDmaPerChunk = PW;                       // transfers that a wave issues per chunk
  // Q8: this lane's share of a chunk on its way through registers
  struct ChunkRegs { u32x4 codes; float2 sz; };
  const bool q8_v = PW == 2 ? lane >= 32 : wave >= 8;     // the lane works on V rows (else K rows)
  const bool q8_active = PW == 2 || lane < 32;
  [[maybe_unused]] auto load_chunk = [&](int tok) -> ChunkRegs {
    ChunkRegs r;
    r.codes = u32x4{0u, 0u, 0u, 0u}; r.sz = make_float2(0.f, 0.f);
    if (q8_active) {
      tok = checked_index(a.hdr, tok, a.kv_len);
      const unsigned char* base = q8_v ? Vp : Kp;
      const float2* sz = (q8_v ? a.v_sz : a.k_sz) + (int64_t)(b * a.H + h) * (a.ks[1] / a.ks[2]);
      r.codes = *(const u32x4*)(base + __umul24((unsigned)tok, row_bytes) + 16u * ((unsigned)lane & 3u));
      r.sz = sz[tok];
    }
    return r;
  };
  [[maybe_unused]] auto commit_chunk = [&](int t, const ChunkRegs& r) {   // chunk t -> ring slots (t % 5) * 64 ...
    if (!q8_active) return;
    const unsigned slot = (unsigned)((t % kRingChunks) * C + row);
    const unsigned sw = ring_swizzle((unsigned)row), p2 = 2u * ((unsigned)lane & 3u);
    unsigned char* dst = (q8_v ? Vring : Kring) + slot * kRingRowBytes;
    bf16x8 lo, hi;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int8_t c0 = (int8_t)((r.codes[e >> 2] >> (8 * (e & 3))) & 0xffu);
      const int8_t c1 = (int8_t)((r.codes[2 + (e >> 2)] >> (8 * (e & 3))) & 0xffu);
      lo[e] = (__bf16)fmaf(r.sz.x, (float)c0, r.sz.y);
      hi[e] = (__bf16)fmaf(r.sz.x, (float)c1, r.sz.y);
    }
    *(bf16x8*)(dst + ((p2 ^ sw) << 4)) = lo;
    *(bf16x8*)(dst + (((p2 + 1u) ^ sw) << 4)) = hi;
  };  // (tokens and descriptors through buffer loads: a scalar resource and a scalar offset plus a
  // lane offset register, where a flat address costs 64-bit vector arithmetic per load)
  const __amdgpu_buffer_rsrc_t tok_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)utok, 0, NC * C * 4, kBufferFlags);
  // the list entry of this lane's row of chunk t (clamped to the last chunk)
  auto load_tok = [&](int t) -> int {
    const int tc = min(t, NC - 1);
    return (int)__builtin_amdgcn_raw_buffer_load_b32(tok_rsrc, row * 4, tc * C * 4, 0);
  };
  // ---- prologue, scalar part.  Everything that comes through scalar loads (patch
  // descriptors, phase tables, the extent of the group's steps) is fetched before the first
  // vector memory operation: behind the burst of first chunks of all workgroups a scalar
  // miss would take microseconds, and the vector loads below depend on these values.
  // Patch descriptor words: {step_begin, n_steps, q_base, sk | ny << 16, nx | kq << 16, pairs, valid, first_ends}
  // (wide patches: {.., nx | kq << 16, ceil(65536 / nx), ..})
  constexpr int kPerGroup = kGroupPatches / PW;          // patches of the list that this form walks
  const WaveDesc* const patches = (WIDE ? wide.waves : a.waves) + grp_g * kPerGroup;
  const const_i32_ptr wA = (const_i32_ptr)(patches + wave);
  const const_i32_ptr wF = (const_i32_ptr)patches, wL = (const_i32_ptr)(patches + kPerGroup - 1);
  const const_i32_ptr pe = (const_i32_ptr)(a.phase_end + gd.phase_base + wave * NC);
  auto last_chunk = [&](int ph) -> int { return min(2 * ph, NC - 1); };   // of phase ph (clamped)
  struct PatchWords { int step_begin, q_base, sk_ny, nx_kq, magic, valid; };   // (the wide patches' band has sk = 0)
  const PatchWords pw = {wA[0], wA[2], wA[3], WIDE ? wA[4] : 0, WIDE ? wA[5] : 0, wA[6]};
  const int first_step = wF[0], n_group_steps = wL[0] + wL[1] - first_step;
  const int last = max(wA[1] - 1, 0);                    // last step of the patch
  // cumulative step counts of phases 0 and 1 (an idle patch has zeros); the entry of
  // phase p + 2 is fetched during phase p
  // (those of phases 0 and 1 sit in the patch descriptor, so that nothing the first vector
  // loads depend on waits for a second round of scalar loads behind the group descriptor)
  const unsigned fe = (unsigned)wA[7];
  int end = (int)(fe & 0xffffu), end1 = (int)(fe >> 16);
  asm volatile("" : : "s"(pw.step_begin), "s"(pw.q_base), "s"(pw.sk_ny), "s"(pw.nx_kq), "s"(pw.magic), "s"(pw.valid),
               "s"(n_group_steps), "s"(end), "s"(end1), "s"(last),
               "s"(gd.union_base), "s"(gd.n_phases), "s"(gd.k), "s"(gd.phase_base), "s"(gd.ident));   // all in
  asm volatile("" : "+s"(c));                            // (so that no step waits for it)
  // Scalar round trip 3, only with an output sharing table: the flag of (head, query scale),
  // as the aligned word that holds the byte (a naturally aligned word lies in its byte's page).
  bool shared = false;
  if (a.cfg_share) {
    const uintptr_t sa = (uintptr_t)(a.cfg_share + h * a.n_scales + gd.k);
    const uint32_t share_word = (uint32_t)*(const_i32_ptr)(sa & ~(uintptr_t)3);
    shared = ((share_word >> (8u * (uint32_t)(sa & 3))) & 0xffu) != 0;
  }
  if (shared && b >= a.B / 2) return;      // the conditional workgroup writes this row

  // ---- prologue, vector part.  The key list usually starts with whole key scales (token =
  // position): the transfers of the first three chunks then wait for no token.
  const bool in_prefix = (min(2, NC - 1) + 1) * C <= gd.ident;

  // Step descriptors: 8 bytes per lane; wide patches 16, the mask included.
  using Desc = std::conditional_t<WIDE, u32x4, uint2>;
  constexpr int kDescLane = WIDE ? kWideDesc : 8, kDescBytes = 64 * kDescLane;
  const unsigned char* const step_desc = (const unsigned char*)a.step_addr;
  const __amdgpu_buffer_rsrc_t desc_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(step_desc + (int64_t)pw.step_begin * kDescBytes), 0, wA[1] * kDescBytes, kBufferFlags);   // (an idle patch's reads give zeros)
  const int lane_desc = lane * kDescLane;
  auto load_desc = [&](int s) -> Desc {
    if constexpr (WIDE) {
      return __builtin_amdgcn_raw_buffer_load_b128(desc_rsrc, lane_desc, s * kDescBytes, 0);
    } else {
      const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(desc_rsrc, lane_desc, s * kDescBytes, 0);
      return make_uint2(v.x, v.y);
    }
  };
  [[maybe_unused]] const uint64_t* masks = a.step_mask + (int64_t)pw.step_begin * 8;

  // local query row of this lane's query column (-1 = none)
  auto query_row = [&](int n, bool clamped) -> int {
    const int sk = pw.sk_ny & 0xffff;
    int dy = n >> 2, dx = n & 3;
    if constexpr (WIDE) { dy = (n * pw.magic) >> 16; dx = n - dy * (pw.nx_kq & 0xffff); }
    const int r = pw.q_base + dy * sk + dx;
    if (clamped) return max(min(r, a.q_len - 1), 0);
    return ((pw.valid >> n) & 1) ? r : -1;
  };
  // The loads go out in the order in which their results are needed: tokens (the transfers of the first three chunks
  // wait for them), step descriptors, Q.  The transfers follow (a load issued behind a chunk is held up until the
  // chunk's data is in), and what needs no memory is formed behind them.
  int tok0 = load_tok(0), tok1 = load_tok(1), tok2 = load_tok(2);
  // Step descriptors for one phase: the first step's is fetched during the phase
  // before (d0), those of the next kLater steps at the start of the phase (dl).
  // (Every register that a vector load fills is used only behind an explicit wait for all
  // of the wave's loads: with chunks in flight the compiler would otherwise place such a wait,
  // the chunks included, before the use.  That also allows loads under uniform conditions,
  // whose number the compiler cannot know: only the descriptors that the phase needs.)
  Desc d0 = load_desc(0), dl[kLater];
#pragma unroll
  for (int i = 0; i < kLater; ++i) dl[i] = Desc{};
  auto load_later = [&](int first, int end) {
#pragma unroll
    for (int i = 0; i < kLater; ++i)
      if (first + 1 + i < end) dl[i] = load_desc(first + 1 + i);
  };
  load_later(0, end);                                   // (phase 0 has no wait of its own before their use)
  // Q rows are loaded unconditionally, from a clamped row where the lane has no query: such
  // a column of S^T holds scores of some other query and is never stored, and MFMA columns do not mix
  constexpr int kQPieces = WIDE ? 4 : 2;
  u32x4 q_raw[kQPieces];                                // 16-byte pieces of the lane's query; Q8: 16 codes each
  [[maybe_unused]] float2 q_sz = make_float2(0.f, 0.f);
  {
    const int ld_row = query_row(n, true);
    const unsigned char* qp = (const unsigned char*)a.q + (b * a.qs[0] + h * a.qs[1] + ld_row * a.qs[2]) * kElem;
    if constexpr (Q8) {
      q_sz = a.q_sz[(int64_t)(b * a.H + h) * a.q_len + ld_row];
      if constexpr (WIDE) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {                   // dims 16 t + 8 hi .. + 7
          const u32x2 r = *(const u32x2*)(qp + 16 * t + 8 * hi);
          q_raw[t >> 1][2 * (t & 1)] = r.x; q_raw[t >> 1][2 * (t & 1) + 1] = r.y;
        }
      } else {
        q_raw[0] = *(const u32x4*)(qp + 16 * hi);
      }
    } else {
#pragma unroll
      for (int t = 0; t < kQPieces; ++t) q_raw[t] = *(const u32x4*)(qp + (WIDE ? 32 * t + 16 * hi : 32 * hi + 16 * t));
    }
  }
  // All workgroups walk the same plan in lock-step, so each phase's first access to its part
  // of the plan would be an HBM miss on every workgroup's critical path.  The workgroups of
  // one XCD (they share an L2) therefore touch the group's step descriptors and lane masks
  // once, each its own slice of the 128-byte lines, while the first chunks are on their way.
  int tokn0 = load_tok(3), tokn1 = load_tok(4);         // tokens of the chunks issued in phase 1
  int warm = 0;
  {
    const char* da = (const char*)step_desc + (int64_t)first_step * kDescBytes;
    const char* ma = (const char*)(a.step_mask + (int64_t)first_step * 8);
    // one load per thread: workgroup `me` of this group on this XCD touches the lines
    // [me T, me T + T), T = threads per workgroup (the workgroups beyond the plan's end all
    // touch its last line; with more lines than workgroups x T the rest is touched in part
    // only, which costs nothing but speed)
    const int lines_d = n_group_steps * (kDescBytes / 128), lines = lines_d + (WIDE ? 0 : (n_group_steps + 1) / 2);
    const int l = min(me * (kGroupPatches / PW * 64) + tid, lines - 1);
    const char* src = WIDE || l < lines_d ? da + (int64_t)l * 128 : ma + (int64_t)(l - lines_d) * 128;
    warm = *(const int*)src;
  }
  int t0 = row, t1 = min(1, NC - 1) * C + row, t2 = min(2, NC - 1) * C + row;
  if (!in_prefix) { t0 = tok0; t1 = tok1; t2 = tok2; }   // (waits for the tokens only)
  asm volatile("" : "+v"(t0), "+v"(t1), "+v"(t2));      // (all three formed before the first transfer)
  if constexpr (Q8) {
    // through registers: the three chunks are requested together, converted and written, and
    // the first barrier finds all of them in the ring
    const ChunkRegs c0 = load_chunk(t0), c1 = load_chunk(t1), c2 = load_chunk(t2);
    commit_chunk(0, c0); commit_chunk(1, c1); commit_chunk(2, c2);
  } else {
    issue_chunk(0, row_at(t0)); issue_chunk(1, row_at(t1)); issue_chunk(2, row_at(t2));
  }
  __builtin_amdgcn_sched_barrier(0);

  std::conditional_t<WIDE, WidePatchState, PatchState> ps;
  [[maybe_unused]] const uint64_t queries = (uint64_t)(unsigned)pw.valid * 0x100000001ull;   // wide: the lanes that hold a query
  [[maybe_unused]] const bool band = (pw.sk_ny & 0xffff) == 0;
  [[maybe_unused]] const float slack = kSlack / c;
  [[maybe_unused]] bf16x8 ones;
  ps.negm = 0.f;
  if constexpr (WIDE) {
    ps.L = 0.f; ps.unset = queries; ps.far = 0;
    const int nx = pw.nx_kq & 0xffff, ny = pw.sk_ny >> 16, dy = (n * pw.magic) >> 16, dx = n - dy * nx;
    const int i0 = (band ? n : dy) - 8 * hi, i1 = (band ? n : ny + dx) - 8 * hi;
#pragma unroll
    for (int e = 0; e < 8; ++e) ps.b[e] = (__bf16)(((int)(i0 == e) | (int)(i1 == e)) ? kMaskB : 0.0f);
    ps.O[0] = f32x16{}; ps.O[1] = f32x16{};
  } else {
    ps.thr = kFloor;
    ps.Lacc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) ps.O[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.0f;
    asm volatile("" : "+v"(ones));   // kept in four registers (the compiler would rebuild it in every step)
  }
  // everything older than chunks 1 and 2 is in: Q, the descriptors and tokens, chunk 0 (Q8: all three chunks)
  if constexpr (Q8) wait_vmcnt<0>(); else wait_vmcnt<2 * kDmaPerChunk>();
#pragma unroll
  for (int t = 0; t < kQPieces; ++t) {
    bf16x8 piece;
    if constexpr (Q8) {
      const unsigned w0 = q_raw[t >> 1][2 * (t & 1)], w1 = q_raw[t >> 1][2 * (t & 1) + 1];
#pragma unroll
      for (int e = 0; e < 8; ++e) piece[e] = (__bf16)fmaf(q_sz.x, (float)(int8_t)(((e < 4 ? w0 : w1) >> (8 * (e & 3))) & 0xffu), q_sz.y);
    } else {
      piece = __builtin_bit_cast(bf16x8, q_raw[t]);
    }
    if constexpr (WIDE) ps.q[t] = piece;
    else if (t == 0) ps.qb0 = piece;
    else ps.qb1 = piece;
  }
  if constexpr (Q8) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // (the ring writes above are visible)
  else asm volatile("s_barrier" ::: "memory");
  asm volatile("" : : "v"(tok0), "v"(tok1), "v"(tok2));   // (their registers stay theirs until here: no wait before another use)

  // One step: 32 keys against the patch's 16 queries.
  [[maybe_unused]] auto run_step16 = [&](auto& ps, const uint2 cur, int s) {
    // lane masks of the step (a scalar load): requested ahead of the K pieces so that the
    // two latencies overlap
    const const_u64_ptr mkp = (const_u64_ptr)((const char*)masks + (unsigned)s * 64u);
    uint64_t mk[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) mk[e] = mkp[e];
    u32x4 k00, k01, k10, k11;
    constexpr int kRingBytes = R * kRingRowBytes;       // (descriptor offsets are relative to either ring)
    lds_read_k_issue(lds_addr(Kring + checked_index(a.hdr, cur.x & 0xffffu, kRingBytes)),
                     lds_addr(Kring + checked_index(a.hdr, cur.x >> 16, kRingBytes)), k00, k01, k10, k11);
    // addresses of the V^T pieces: computed while the K pieces are on their way
    unsigned v0 = lds_addr(Kring + checked_index(a.hdr, cur.y & 0xffffu, kRingBytes)),
             v1 = lds_addr(Kring + checked_index(a.hdr, cur.y >> 16, kRingBytes));
    unsigned va_addr[3][2];
#pragma unroll
    for (int dt = 1; dt < 4; ++dt) { va_addr[dt - 1][0] = v0 ^ (32u * dt); va_addr[dt - 1][1] = v1 ^ (32u * dt); }
    asm volatile("" : "+v"(v0), "+v"(v1), "+v"(va_addr[0][0]), "+v"(va_addr[0][1]), "+v"(va_addr[1][0]),
                 "+v"(va_addr[1][1]), "+v"(va_addr[2][0]), "+v"(va_addr[2][1]));
    lds_wait_k(k00, k01, k10, k11);
    // (the masks were requested before the K pieces and share their counter: they are in,
    // and the compiler should know before the V^T reads go out, or it waits for those too)
    asm volatile("" : : "s"(mk[0]), "s"(mk[1]), "s"(mk[2]), "s"(mk[3]), "s"(mk[4]), "s"(mk[5]), "s"(mk[6]), "s"(mk[7]));
    // The accumulators of the score tiles start at -m where the pair is kept and at -inf
    // where it is not (one v_cndmask per score, by the lane masks, off the path that waits
    // for the matrix pipe): the tiles come out as masked scores relative to the reference.
    f32x4 S0, S1;
#pragma unroll
    for (int e = 0; e < 4; ++e) { S0[e] = mask_select(ps.negm, mk[e]); S1[e] = mask_select(ps.negm, mk[4 + e]); }
    S0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k00), ps.qb0, S0, 0, 0, 0);
    S1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k10), ps.qb0, S1, 0, 0, 0);
    S0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k01), ps.qb1, S0, 0, 0, 0);
    S1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k11), ps.qb1, S1, 0, 0, 0);

    // V^T operands: issued behind the score MFMAs, consumed after the exponentials
    uint2 va[4][2];
    lds_read_v<VOFF>(v0, v1, va_addr, va);
    float sv[8] = {S0[0], S0[1], S0[2], S0[3], S1[0], S1[1], S1[2], S1[3]};
    // The reference m of a query only moves when one of its scores exceeds it by more than
    // the slack (probabilities stay below 2^kSlack), and once at the query's first kept key.
    // The common case needs the lane's own maximum only; the maximum over the query's four
    // lanes is formed when some lane of the wave has crossed its threshold.
    const float m012 = fmaxf(fmaxf(sv[0], sv[1]), sv[2]), m345 = fmaxf(fmaxf(sv[3], sv[4]), sv[5]);   // (v_max3)
    const float mx = fmaxf(fmaxf(fmaxf(sv[6], sv[7]), m012), m345);
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(mx > ps.thr) != 0, 0)) {   // rare after the first steps
      const float mxr = max_across_rows(mx);
      const bool grow = mxr > ps.thr;
      const float shift = grow ? mxr : 0.f;               // m moves by this much (down only when m was unset)
      const float alpha = __builtin_amdgcn_exp2f(-fmaxf(shift, 0.f) * c);
      ps.negm -= shift;
      ps.thr = grow ? slack : ps.thr;
#pragma unroll
      for (int e = 0; e < 8; ++e) sv[e] -= shift;
      ps.Lacc *= alpha;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) ps.O[dt] *= alpha;
    }
    float p[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) p[e] = __builtin_amdgcn_exp2f(sv[e] * c);
    bf16x8 pb;
#pragma unroll
    for (int e = 0; e < 8; ++e) pb[e] = (__bf16)p[e];

    lds_wait(va);
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) {
      const uint4 v8 = {va[dt][0].x, va[dt][0].y, va[dt][1].x, va[dt][1].y};
      ps.O[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(v8), pb, ps.O[dt], 0, 0, 0);
    }
    ps.Lacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pb, ps.Lacc, 0, 0, 0);
  };

  // One step of a wide patch: 32 keys against 32 queries.  The arithmetic is that of a 16-query step; what differs:
  //  * The mask is a matrix product too.  A window is a product of rows and columns: dimension i < ny of it stands for
  //    query row i, dimension ny + j for query column j; the B operand has a two where the query lies in that
  //    row or column, the A operand -2^127 or more where the key is not kept by it (else zero or a subnormal), from the
  //    descriptor's sixteen bits per lane.  Their products pass the range of fp32, so the score tile starts at -inf where
  //    the key is not kept and below 2^-123 elsewhere, with seven vector instructions, where sixteen selects took a
  //    scalar load of 128 bytes per step on the wave's critical path.  Bands take two products with one dimension per
  //    query.  (With ones for the twos a raw product of 2^127, or a softmax scale of 1e-37, let masked keys through.)
  //  * The row sums are the lane's own (v_dot2 on the rounded probabilities; a product with ones would need
  //    sixteen more registers).
  //  * No maximum is formed.  The softmax reference starts at zero and moves only when a query's sum leaves
  //    [2^-10, 2^40] (the lower end is looked at until every query has passed it), which costs one comparison
  //    where the maximum of sixteen scores costs eight.  Probabilities and sums keep their relative precision
  //    under any common factor, and the factors are powers of two; the products with V do from sums of 2^-10 on.
  [[maybe_unused]] auto run_step32 = [&](auto& ps, const u32x4 cur) {
    constexpr int kRingBytes = R * kRingRowBytes;
    u32x4 kr[4];
    lds_read_k_row_issue(lds_addr(Kring + checked_index(a.hdr, cur.x, kRingBytes)), kr);
    unsigned v[4] = {cur.y & 0xffffu, cur.y >> 16, cur.z & 0xffffu, cur.z >> 16}, x[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[i] = lds_addr(Kring + checked_index(a.hdr, v[i], kRingBytes));
      x[i] = v[i] ^ 64u;
    }
    const unsigned mask_bits = cur.w;          // (a bit cast of a vector's element would read element 0)
    // 16-bit halves of the descriptor's mask word: bits 15, 13, .. are elements 0, 2, .. (low half) or 1, 3, .. (high half);
    // moved to the sign and spread over eight bits, a set one reads as bf16 -2^127 or up to twice that
    auto mask_operand = [&](int first) -> bf16x8 {
      u32x4 m;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const s16x2 bits = __builtin_bit_cast(s16x2, mask_bits) << (short)(2 * (first + r));
        m[r] = __builtin_bit_cast(unsigned, bits >> (short)7);
      }
      return __builtin_bit_cast(bf16x8, m);
    };
    f32x16 S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(mask_operand(0), ps.b, f32x16{}, 0, 0, 0);
    if (band) {
      int i = n - 16 - 8 * hi;                           // (formed here: not worth four registers of every plan)
      asm volatile("" : "+v"(i));
      bf16x8 upper;
#pragma unroll
      for (int e = 0; e < 8; ++e) upper[e] = (__bf16)(i == e ? kMaskB : 0.0f);
      S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(mask_operand(4), upper, S, 0, 0, 0);
    }
    asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]));
    lds_wait_k(kr[0], kr[1], kr[2], kr[3]);
#pragma unroll
    for (int t = 0; t < 4; ++t)
      S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kr[t]), ps.q[t], S, 0, 0, 0);
    u32x2 va[8];
    lds_read_v_wide<VOFF>(v, x, va);
    __builtin_amdgcn_sched_barrier(0);         // (the reads go out here, not behind the exponentials)
    bf16x8 pb[2];
    float sum;
    auto exponentials = [&]() {
      sum = ps.L;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
#pragma unroll
        for (int e = 0; e < 8; ++e) pb[t][e] = (__bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(S[8 * t + e], c, ps.negm));
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
          const bf16x2 two = {pb[t][e], pb[t][e + 1]};
          sum = __builtin_amdgcn_fdot2_f32_bf16(two, kOnes, sum, false);
        }
      }
    };
    exponentials();
    uint64_t move = __builtin_amdgcn_ballot_w64(sum > kMostSum);
    if (__builtin_expect(ps.unset != 0, 0)) {
      ps.unset = __builtin_amdgcn_ballot_w64(sum + other_half(sum) < kLeastSum) & queries;
      move |= ps.unset;
    }
    if (__builtin_expect(move != 0, 0)) {
      float mx = S[0];
#pragma unroll
      for (int e = 1; e < 16; ++e) mx = fmaxf(mx, S[e]);
      mx = fmaxf(mx, other_half(mx));                    // over both lanes of the query
      const float now = sum + other_half(sum), before = ps.L + other_half(ps.L);
      float to = mx > -INFINITY ? __builtin_fmaf(mx, c, ps.negm) : kFloor;
      if (before > 0.f) to = fmaxf(to, __builtin_amdgcn_logf(before));         // (base 2)
      const float shift = (now > kMostSum || now < kLeastSum) && to > kFloor ? rintf(to) : 0.f;
      const float alpha = before > 0.f ? __builtin_amdgcn_exp2f(-shift) : 1.f;
      ps.negm -= shift; ps.L *= alpha;
      ps.far |= is_far(ps.negm);
#pragma unroll
      for (int e = 0; e < 16; ++e) { ps.O[0][e] *= alpha; ps.O[1][e] *= alpha; }
      exponentials();
      if (ps.unset) ps.unset = __builtin_amdgcn_ballot_w64(sum + other_half(sum) < kLeastSum) & queries;
    }
    ps.L = sum;
    lds_wait_v_wide(va);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int dt = 0; dt < 2; ++dt) {
        const uint4 v8 = {va[4 * t + dt].x, va[4 * t + dt].y, va[4 * t + 2 + dt].x, va[4 * t + 2 + dt].y};
        ps.O[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(v8), pb[t], ps.O[dt], 0, 0, 0);
      }
  };
  auto run_step = [&](const Desc cur, int s) {
    if constexpr (WIDE) run_step32(ps, cur); else run_step16(ps, cur, s);
  };

  // ---- phases ----
  int done = 0;                                         // steps finished so far
  // (phase 0 is a copy of its own: of a condition that stands twice the compiler also considers the mixed paths, on
  // which it would have to wait for loads that are long in)
  auto run_phase = [&](int ph, auto is_first) -> bool {
    constexpr bool FIRST = decltype(is_first)::value;
    const bool next = ph + 1 < P;                        // (P >= 1; a list of one chunk has no steps after phase 0)
    if (!FIRST && ph == kBoostPhases) __builtin_amdgcn_s_setprio(0);
    [[maybe_unused]] ChunkRegs cr0{}, cr1{};             // Q8: the chunks of phase ph + 1 on their way
    const int end2 = pe[last_chunk(ph + 2)];            // (a scalar load, two phases ahead of its use)
    if constexpr (!FIRST) load_later(done, end);        // (phase 0: fetched in the prologue)
    if (done < end) run_step(d0, done);
    // The later descriptors have had a step to arrive; with nothing else outstanding
    // when the chunks go out, no later use of a loaded register has to wait for them
    // (the compiler would otherwise wait for everything, the chunks included).
    if constexpr (!FIRST) wait_vmcnt<0>();
    if (next) {
      // first descriptor and tokens of the next phase: in place, their users are done
      // (ahead of the chunks: a load issued behind a chunk is held up until its data is in)
      d0 = load_desc(min(end, last));
      if constexpr (!FIRST) {
        [[maybe_unused]] unsigned r0 = 0, r1 = 0;
        if constexpr (Q8) { cr0 = load_chunk(tokn0); cr1 = load_chunk(tokn1); }
        else { r0 = row_at(tokn0); r1 = row_at(tokn1); asm volatile("" : "+v"(r0), "+v"(r1)); }   // (formed before the registers are loaded again)
        tokn0 = load_tok(2 * ph + 3); tokn1 = load_tok(2 * ph + 4);
        // the chunks of phase ph + 1, into the slots of chunks 2 ph - 4 and 2 ph - 3
        if constexpr (!Q8) { issue_chunk(2 * ph + 1, r0); issue_chunk(2 * ph + 2, r1); }
      }
    }
#pragma unroll
    for (int i = 0; i < kLater; ++i)
      if (done + 1 + i < end) run_step(dl[i], done + 1 + i);
    // (a patch rarely has more steps in a phase; their descriptors are loaded on the spot)
    for (int s = done + 1 + kLater; s < end; ++s) run_step(load_desc(s), s);
    done = end;
    end = end1; end1 = end2;
    // The chunks of phase ph + 1, the next descriptors and tokens are in once nothing of
    // this wave is outstanding.  All LDS reads of the phase have returned (each step waits
    // for its own), so after the barrier the slots of chunks 2 ph - 3 and 2 ph - 2 are free.
    wait_vmcnt<0>();
    if (!next) return false;
    if constexpr (Q8 && !FIRST) {
      // (their slots held chunks 2 ph - 4 and 2 ph - 3, which nobody has read since the
      // barrier that ended phase ph - 1; the writes are complete before this phase's barrier)
      commit_chunk(2 * ph + 1, cr0); commit_chunk(2 * ph + 2, cr1);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    asm volatile("s_barrier" ::: "memory");
    return true;
  };
  if (run_phase(0, std::true_type{})) {
    int ph = 1;
    while (run_phase(ph, std::false_type{})) ++ph;
  }

  asm volatile("" : : "v"(warm));      // the only use of the plan-touching load: keeps it

  // ---- epilogue ----
  int n_again = n;                             // recomputed from scratch: the row is not worth a
  asm volatile("" : "+v"(n_again));            // register (or a spill slot) through the loop
  int qrow = query_row(n_again, false);
  if constexpr (WIDE) {
    const float sum = ps.L + other_half(ps.L), inv = 1.f / sum;
    float any = 0.f;
    unsigned r[2][8];
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
      for (int e = 0; e < 16; e += 2) {
        const bf16x2 two = {(__bf16)(ps.O[dt][e] * inv), (__bf16)(ps.O[dt][e + 1] * inv)};
        any = __builtin_amdgcn_fdot2_f32_bf16(two, kOnes, any, false);
        r[dt][e / 2] = __builtin_bit_cast(unsigned, two);
      }
    // A matrix product multiplies the rows of a step with the probability 0 of the queries that do not keep them, so a
    // value that is not finite makes all queries of its step NaN: in every dimension where it is K's, in its own where
    // it is V's.  Those dimensions are formed once more behind the store, query by query, from the kept pairs alone;
    // rows whose reference went too far in all dimensions.
    const float rest_of_row = other_half(any);
    const bool far = __builtin_amdgcn_inverse_ballot_w64(ps.far);
    const bool bad = qrow >= 0 && (not_finite(any) || not_finite(rest_of_row) || far);
    const unsigned rows_again = (unsigned)__builtin_amdgcn_ballot_w64(bad);
    unsigned bad_dims = 0;
    if (__builtin_expect(rows_again != 0, 0)) bad_dims = far || not_finite(sum) ? ~0u : not_finite_dims(r);
    if (qrow >= 0) {
      const int to = checked_index(a.hdr, qrow, a.q_len);
      __bf16* op = (__bf16*)a.o + b * a.os[0] + h * a.os[1] + to * a.os[2] + 8 * hi;
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
    attend_rows<Q8>(a, c, b, h, shared, rows_again, qrow, bad_dims,
                    [&](int row) { return StepKeys(a, a.waves + (size_t)grp_g * kGroupPatches, row); });
  } else {
    if (qrow < 0) return;
    qrow = checked_index(a.hdr, qrow, a.q_len);
    const float inv = 1.f / ps.Lacc[0];
    __bf16* op = (__bf16*)a.o + b * a.os[0] + h * a.os[1] + qrow * a.os[2] + 4 * hi;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) {
      bf16x4 r;
#pragma unroll
      for (int i = 0; i < 4; ++i) r[i] = (__bf16)(ps.O[dt][i] * inv);
      *(bf16x4*)(op + 16 * dt) = r;
      if (shared) *(bf16x4*)(op + (a.B / 2) * a.os[0] + 16 * dt) = r;
    }
  }
}

litevar_status launch_attn_bf16_pair(const litevar_plan* pl, const AttnArgs& args, hipStream_t st) {
  if (pl->waves_per_group != 16 || pl->chunk_keys != kDmaKeys || pl->ring_chunks != kRingChunks)
    return fail(LITEVAR_E_PLAN_CORRUPT, "no 16-patch kernel for chunk=%d ring=%d", pl->chunk_keys, pl->ring_chunks);
  AttnArgs a = args;
  const int64_t blocks = spread_over_xcds(a, a.n_groups, a.k_sz ? 72 : 128);
  if (blocks > 0x7fffffff) return fail(LITEVAR_E_UNSUPPORTED, "grid too large");
  // Sixteen waves with a 16-query patch each where the plan asks for them, or can have no wide patches.  They are nowhere
  // quicker, on a CU of their own either: 256 queries on 680 keys, 60 / 240 pairs 14.0 / 17.0 us, wide 13.4 / 16.4; 169
  // queries 10.5 / 11.6, wide 10.4 / 11.6; 1024 on 2240 keys, 60 pairs 22.8, wide 21.2; 680 tokens, 8 pairs 12.7, wide 12.1.
  const int64_t groups = (int64_t)pl->n_groups * pl->n_head_groups;
  // (A plan has wide patches where its section of patches holds theirs: a group's 16 descriptors are 512 bytes and its
  // eight wide ones 256, so the section has no padding.)
  const bool has_wide = pl->off[kSecPhaseEnd] - pl->off[kSecWaves] == (uint64_t)groups * (16 + kWidePatches) * sizeof(WaveDesc);
  if ((has_wide && pl->patches_per_wave == 1) || pl->off[kSecStepAddr] - pl->off[kSecUnion] != (uint64_t)pl->n_union_keys * sizeof(int32_t))
    return fail(LITEVAR_E_PLAN_CORRUPT, "the plan's sections are not those of this library");
  const int pw = has_wide ? 2 : 1;
  WideArgs w{};
  w.waves = a.waves + groups * 16;
  // all workgroups are resident at once (two per CU): see later_arrival
  static thread_local int n_cu[64] = {0};
  int dev = 0;
  if (litevar_status s = hip_check(hipGetDevice(&dev), "hipGetDevice")) return s;
  if (dev >= 0 && dev < 64 && n_cu[dev] == 0)
    if (litevar_status s = hip_check(hipDeviceGetAttribute(&n_cu[dev], hipDeviceAttributeMultiprocessorCount, dev),
                                     "hipDeviceGetAttribute")) return s;
  w.boost = blocks <= 2 * (dev >= 0 && dev < 64 ? n_cu[dev] : 256);
  const float c = a.sm_scale * 1.4426950408889634f;
  const bool q8 = a.k_sz != nullptr;
  const dim3 wg(kGroupPatches / pw * 64);
  return launch_in_parts(blocks, (int)wg.x, "bf16 attention launch", [&](int64_t first, unsigned n) {
    a.first_block = (uint32_t)first;
    if (pw == 1 && q8) hipLaunchKernelGGL((k_attn_bf16_pair<1, true>), dim3(n), wg, 0, st, a, w, c);
    else if (pw == 1) hipLaunchKernelGGL((k_attn_bf16_pair<1, false>), dim3(n), wg, 0, st, a, w, c);
    else if (q8) hipLaunchKernelGGL((k_attn_bf16_pair<2, true>), dim3(n), wg, 0, st, a, w, c);
    else hipLaunchKernelGGL((k_attn_bf16_pair<2, false>), dim3(n), wg, 0, st, a, w, c);
  });
}

}  // namespace lv
