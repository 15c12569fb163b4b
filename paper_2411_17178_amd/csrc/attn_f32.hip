// fp32 windowed attention forward: the accuracy path (1e-5 against the fp64 oracle).
// Section 2 of the paper: softmax over the kept keys only.  fp32 operands, products, sums and
// exponentials throughout.
//
// One workgroup = four waves (one, where every patch has a single step) = one query patch of one
// (batch, head); wave w takes the patch's 32-key steps w, w + 4, ... (the plan's steps and lane masks, as
// the bf16 kernels walk them) and the four partial results are merged through LDS at the end.  The products run on
// v_mfma_f32_16x16x4_f32, straight from global memory: nothing of K or V is shared between the
// waves of a workgroup, and the operand order can be chosen so that every load is a 16-byte piece
// of a row and no value has to move between lanes:
//   S^T = K Q^T   contraction slice (j, e) of the head dimension is {16 j + 4 g4 + e : g4 = 0..3},
//                 so lane (n, g4) = (lane % 16, lane / 16) loads floats 16 j + 4 g4 .. + 3 of row n
//                 (four lanes cover 64 contiguous bytes); it receives the scores of query n
//                 with the four keys 4 g4 + i of a tile;
//   O^T += V^T P^T  contraction slice i is the keys {4 g4 + i}: the B operand is the lane's own
//                 probability, and row n of dimension tile dt is dimension 4 n + dt, so one
//                 16-byte load of V's row feeds all four tiles (sixteen lanes cover a row).
//
// Bound: a step is 64 MFMAs of 32 cycles (2048 cycles of a SIMD's matrix pipe) against 16 KB of
// gathered rows; four waves per patch, because the accuracy workloads have few patches (57 per
// (batch, head) at 680 tokens) and the longest one would otherwise be a chain of eleven steps.
// 680 tokens, 32 (batch, head) pairs, radius 2: 29.5 us a call (one wave per patch with scalar dot
// products and a shuffle per key: 233 us); the matrix pipe's share is 8 us, the rest is the chain
// descriptor -> tokens -> rows -> MFMAs of two rounds of workgroups.  (30.1 with the patch's words in three round
// trips and the queries ahead of the first tokens; 2 pairs at radius 4 11.2 -> 11.05.  K rows requested a step
// ahead take 136 registers instead of 99: 31.6.  Steps dealt from another wave in every patch: no change.)
#include "attn_bf16_common.h"

namespace lv {

namespace {

constexpr float kF32Floor = -3.402823466e+38f;   // softmax reference of a query without a kept key so far

}  // namespace

// W = waves per patch, 4 or 1
template <int W>
__global__ __launch_bounds__(W * 64) void k_attn_f32(AttnArgs a, int n_waves) {
  int me, bh, wv, b, h;
  if (!xcd_item(a, n_waves, me, bh, wv)) return;
  divmod_by((uint32_t)bh, (uint32_t)a.H, a.H_magic, b, h);
  const int head_group = a.head_map ? ((const_i32_ptr)a.head_map)[h] : 0;   // (in the header's round trip)
  if (!plan_usable(a.hdr)) return;
  // the patch's words in one scalar load (left alone they come in three round trips, the first for ny)
  const const_u64_ptr wp = (const_u64_ptr)(a.waves + (wv + head_group * n_waves));
  uint64_t w0 = wp[0], w1 = wp[1], w2 = wp[2], w3 = wp[3];
  asm volatile("" : "+s"(w0), "+s"(w1), "+s"(w2), "+s"(w3));
  const uint64_t words[4] = {w0, w1, w2, w3};
  const WaveDesc wd = __builtin_bit_cast(WaveDesc, words);
  if (wd.ny == 0) return;
  const bool shared = a.cfg_share && a.cfg_share[h * a.n_scales + wd.kq];
  if (shared && b >= a.B / 2) return;

  const int lane = threadIdx.x & 63, n = lane & 15, g4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int dy = n >> 2, dx = n & 3;
  const int qrow = ((wd.valid >> n) & 1u) ? checked_index(a.hdr, wd.q_base + dy * wd.sk + dx, a.q_len) : -1;

  const char* Kp = (const char*)((const float*)a.k + b * a.ks[0] + h * a.ks[1]);
  const char* Vp = (const char*)((const float*)a.v + b * a.ks[0] + h * a.ks[1]);
  const unsigned row_bytes = (unsigned)a.ks[2] * 4u;   // (24 bits, and a slab spans < 2 GiB: checked by the API)

  f32x4 qv[4], O[4];
  const float* Q = (const float*)a.q + b * a.qs[0] + h * a.qs[1];
#pragma unroll
  for (int j = 0; j < 4; ++j) { qv[j] = f32x4{0.f, 0.f, 0.f, 0.f}; O[j] = qv[j]; }
  float m = kF32Floor, l = 0.f;          // softmax reference of query n (the same in its four lanes), this lane's row sum

  const int64_t S0 = wd.step_begin;
  const int n_steps = wd.n_steps;
  // the tokens of this lane's K rows (keys n and 16 + n) and V rows (keys 16 t + 4 g4 + i) of a step
  struct Tokens { int k[2]; int4 v[2]; };
  auto load_tokens = [&](int s) {
    const int32_t* t = a.step_tok + (S0 + min(s, n_steps - 1)) * kStepKeys;
    return Tokens{{t[n], t[16 + n]}, {*(const int4*)(t + 4 * g4), *(const int4*)(t + 16 + 4 * g4)}};
  };
  Tokens tok = load_tokens(wave);
  __builtin_amdgcn_sched_barrier(0);         // (the queries behind the tokens, for which the rows wait)
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (qrow >= 0) qv[j] = *(const f32x4*)(Q + qrow * a.qs[2] + 16 * j + 4 * g4);
  for (int s = wave; s < n_steps; s += W) {
    // (padding keys carry token -1; they read the row of the step's first key, which every step has)
    const int first = __builtin_amdgcn_readfirstlane(tok.k[0]);
    auto row = [&](int t) -> unsigned {
      return __umul24((unsigned)checked_index(a.hdr, t < 0 ? first : t, a.kv_len), row_bytes);
    };
    f32x4 kf[2][4], vf[2][4];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const unsigned o = row(tok.k[t]) + 16u * (unsigned)g4;
#pragma unroll
      for (int j = 0; j < 4; ++j) kf[t][j] = *(const f32x4*)(Kp + (o + 64u * j));
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int vt[4] = {tok.v[t].x, tok.v[t].y, tok.v[t].z, tok.v[t].w};
#pragma unroll
      for (int i = 0; i < 4; ++i) vf[t][i] = *(const f32x4*)(Vp + (row(vt[i]) + 16u * (unsigned)n));
    }
    const const_u64_ptr mk = (const_u64_ptr)(a.step_mask + (S0 + s) * 8);
    uint64_t keep[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) keep[e] = mk[e];
    tok = load_tokens(s + W);

    f32x4 S[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int t = 0; t < 2; ++t) S[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[t][j][e], qv[j][e], S[t], 0, 0, 0);

    float z[8], mx = kF32Floor;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      z[e] = mask_select(S[e >> 2][e & 3] * a.sm_scale, keep[e]);
      mx = fmaxf(mx, z[e]);
    }
    const float m_new = fmaxf(m, max_across_rows(mx));
    if (__builtin_amdgcn_ballot_w64(m_new > m) != 0) {
      const float alpha = expf(m - m_new);
      l *= alpha;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) O[dt] *= alpha;
      m = m_new;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) { z[e] = expf(z[e] - m); l += z[e]; }      // (masked: exp(-inf) = 0)
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
        O[dt] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[e >> 2][e & 3][dt], z[e], O[dt], 0, 0, 0);
  }

  // ---- the head dimensions 16 g4 + 4 c .. + 3 of query n, c = 4 / W of 0..3: merged from the four waves, or its own
  constexpr int kPieces = 4 / W;
  f32x4 acc[kPieces];
  float sum = 0.f;
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  if constexpr (W == 4) {
    __shared__ __align__(16) f32x4 part_o[W][4][64];
    __shared__ float part_m[W][16], part_l[W][16];
#pragma unroll
    for (int i = 0; i < 4; ++i) part_o[wave][i][lane] = f32x4{O[0][i], O[1][i], O[2][i], O[3][i]};
    if (g4 == 0) { part_m[wave][n] = m; part_l[wave][n] = l; }
    __syncthreads();
    float m_all = part_m[0][n];
#pragma unroll
    for (int w = 1; w < W; ++w) m_all = fmaxf(m_all, part_m[w][n]);
    acc[0] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const float f = expf(part_m[w][n] - m_all);
      sum = fmaf(part_l[w][n], f, sum);
      acc[0] += part_o[w][wave][lane] * f;
    }
  } else {
    sum = l;
#pragma unroll
    for (int c = 0; c < kPieces; ++c) acc[c] = f32x4{O[0][c], O[1][c], O[2][c], O[3][c]};
  }
  float any = 0.f;
#pragma unroll
  for (int c = 0; c < kPieces; ++c) {
    acc[c] *= 1.f / sum;
    any += (acc[c][0] + acc[c][1]) + (acc[c][2] + acc[c][3]);
  }

  // The matrix products multiply the V rows of a step with the probability 0 of every query that does not
  // keep them, so a value of V that is not finite makes all queries of its step NaN.  A wave that finds such a
  // result forms its head dimensions once more, key by key, from the kept pairs only.  (680 tokens, 32 pairs:
  // the test costs 0.3 us of 30.)
  const bool again = qrow >= 0 && not_finite(any);
  if (__builtin_amdgcn_ballot_w64(again) != 0) {
    m = kF32Floor; l = 0.f;
#pragma unroll
    for (int c = 0; c < kPieces; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int64_t q_at = max(qrow, 0) * a.qs[2] + 4 * g4;   // (Q from memory: its registers are free by now)
    for (int64_t e = S0 * kStepKeys; e < (S0 + n_steps) * kStepKeys; ++e) {
      const int t = a.step_tok[e];
      if (t < 0) continue;                               // padding key (uniform over the wave)
      const unsigned o = __umul24((unsigned)checked_index(a.hdr, t, a.kv_len), row_bytes) + 16u * (unsigned)g4;
      float dot = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 kr = *(const f32x4*)(Kp + (o + 64u * j)), qr = *(const f32x4*)(Q + q_at + 16 * j);
#pragma unroll
        for (int i = 0; i < 4; ++i) dot = fmaf(qr[i], kr[i], dot);
      }
      dot += __shfl_xor(dot, 16);
      dot += __shfl_xor(dot, 32);
      const int r = (int)e & 15;
      const uint64_t keep = a.step_mask[(e >> 5) * 8 + 4 * ((e >> 4) & 1) + (r & 3)] >> ((r >> 2) * 16);
      if ((keep >> n) & 1) {
        const float z = dot * a.sm_scale, m_new = fmaxf(m, z), alpha = expf(m - m_new), p = expf(z - m_new);
        l = fmaf(l, alpha, p);
        m = m_new;
#pragma unroll
        for (int c = 0; c < kPieces; ++c) {
          const f32x4 vr = *(const f32x4*)(Vp + (o + 48u * (unsigned)g4 + 16u * (unsigned)(wave + c)));
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[c][i] = fmaf(p, vr[i], acc[c][i] * alpha);
        }
      }
    }
#pragma unroll
    for (int c = 0; c < kPieces; ++c) acc[c] *= 1.f / l;
  }
  if (qrow < 0) return;
  float* o = (float*)a.o + b * a.os[0] + h * a.os[1] + qrow * a.os[2] + 16 * g4 + 4 * wave;
#pragma unroll
  for (int c = 0; c < kPieces; ++c) {
    *(f32x4*)(o + 4 * c) = acc[c];
    if (shared) *(f32x4*)(o + 4 * c + (a.B / 2) * a.os[0]) = acc[c];
  }
}

litevar_status launch_attn_f32(const litevar_plan* pl, const AttnArgs& args, hipStream_t st) {
  AttnArgs a = args;
  // Patches of one step each leave three of four waves without work, and a launch of many such patches is
  // as long as it takes to start its waves.  Pairs x 14 tokens (scales 1, 2, 3), one wave per patch with scalar
  // dot products / four waves / one wave: 480: 23.3 / 25.6 / 13.5 us; 3000: 119 / 152 / 63; 100 000: 4346 / 6083 /
  // 2125.  (One token per pair: 480: 6.3 / 10.0 / 6.3; 3000: 15.4 / 46.3 / 22.4.)  With more steps four waves shorten
  // the chain of the launch's longest patch: 85 tokens at 8 pairs 5.4 us, 6.4 with one wave.
  const int W = pl->n_steps <= (int64_t)pl->n_patches * pl->n_head_groups ? 1 : 4;
  const int64_t n_waves = (int64_t)pl->n_groups * pl->waves_per_group;
  const int64_t blocks = spread_over_xcds(a, n_waves, 256);
  if (blocks > 0x7fffffff) return fail(LITEVAR_E_UNSUPPORTED, "grid too large for the fp32 path");
  return launch_in_parts(blocks, W * 64, "fp32 attention launch", [&](int64_t first, unsigned n) {
    a.first_block = (uint32_t)first;
    if (W == 1) hipLaunchKernelGGL(k_attn_f32<1>, dim3(n), dim3(64), 0, st, a, (int)n_waves);
    else hipLaunchKernelGGL(k_attn_f32<4>, dim3(n), dim3(256), 0, st, a, (int)n_waves);
  });
}

}  // namespace lv
