// QK-norm, RoPE and the cache write of one head of one row (head_dim 128, bf16, MFMA cache layout), by the sixteen lanes that own the
// head: a kernel of its own for many rows, or the first thing that the decode attention of few rows does.
#pragma once
#include "kernels.h"

// Lane `sub` holds dims 4 sub .. 4 sub + 3 and their rotate-half partners 64 + ..., so partial sums arrive as 16-byte loads (all
// issued before the first add) and q, k leave as 8-byte stores.  q: *w1, *w2 get dims 4 sub .. and 64 + 4 sub .. in bf16.  k, v: written
// to the page that page() names.  FP8: keys and values go from fp32 straight to E4M3 codes (8-bit cache layout).
// UNDIV: the row is still to be divided by the rms of the projection's input, ssq holds that input's sums of squares.  A
// choice at compile time: tested at run time the plain form with the 8-bit cache took 101 registers instead of 84, 4 waves
// a SIMD instead of 5.
template <bool FP8, bool UNDIV, typename F>
__device__ __forceinline__ void qkrope_head128(const RopeArgs& a, int row, int hd, int sub, int pos, F page, bf16_t* __restrict__ kpool,
                                               bf16_t* __restrict__ vpool, uint2* w1, uint2* w2) {
  const int NH = a.nq + 2 * a.nkv;
  const float* x = a.qkv + ((size_t)row * NH + hd) * 128 + sub * 4;
  float4 lo[8], hi[8];
#pragma unroll
  for (int p = 0; p < 8; p++) {
    lo[p] = p < a.n_part ? *(const float4*)(x + (size_t)p * a.part_stride) : make_float4(0.f, 0.f, 0.f, 0.f);
    hi[p] = p < a.n_part ? *(const float4*)(x + (size_t)p * a.part_stride + 64) : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  float sq = 0.f;            // the row's sum of squares where its norm is still to be applied: n16 partial sums
  if (UNDIV)
    for (int x = sub; x < a.n16; x += 16 * 8) {      // eight reads in flight: one at a time cost 2.6 us (160 sums) to 4 us
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; u++) v[u] = a.ssq[min(x + 16 * u, a.n16 - 1) * a.ss_stride + row];
#pragma unroll
      for (int u = 0; u < 8; u++) sq += x + 16 * u < a.n16 ? v[u] : 0.f;
    }
  const bool is_q = hd < a.nq, is_v = hd >= a.nq + a.nkv;
  const bf16_t* g = is_q ? a.gq : a.gk;
  const uint2 glo = *(const uint2*)(g + sub * 4), ghi = *(const uint2*)(g + 64 + sub * 4);
  const float* cs = a.rope_cs + ((size_t)pos * 64 + sub * 4) * 2;     // (cos, sin) pairs of 4 dims
  const float4 cs0 = *(const float4*)cs, cs1 = *(const float4*)(cs + 4);
  float u[4] = {lo[0].x, lo[0].y, lo[0].z, lo[0].w}, w[4] = {hi[0].x, hi[0].y, hi[0].z, hi[0].w};
#pragma unroll
  for (int p = 1; p < 8; p++)
    if (p < a.n_part) {
      u[0] += lo[p].x; u[1] += lo[p].y; u[2] += lo[p].z; u[3] += lo[p].w;
      w[0] += hi[p].x; w[1] += hi[p].y; w[2] += hi[p].z; w[3] += hi[p].w;
    }
  if (UNDIV) {
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 16);
    const float inv = 1.0f / sqrtf(sq / (float)a.hidden + a.eps);
#pragma unroll
    for (int e = 0; e < 4; e++) { u[e] *= inv; w[e] *= inv; }
  }
  // fused multiply-adds as written, here and in the rotation: left to the compiler, which of two products it rounds differs from kernel to
  // kernel, and with it a key's last bit
  float ss = 0.f;
#pragma unroll
  for (int e = 0; e < 4; e++) ss += __builtin_fmaf(u[e], u[e], w[e] * w[e]);
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 16);
  const int tok = pos & (RL_PAGE - 1);
  bf16_t* blk = nullptr;
  uint8_t* blk8 = nullptr;
  if (!is_q) {
    const size_t at = ((size_t)page() * a.nkv + (is_v ? hd - a.nq - a.nkv : hd - a.nq)) * (RL_PAGE * 128);
    blk = (is_v ? vpool : kpool) + at;
    blk8 = (uint8_t*)(is_v ? vpool : kpool) + at;
  }
  if (is_v) {
#pragma unroll
    for (int e = 0; e < 4; e++) {
      if constexpr (FP8) {
        blk8[vswz8_off(tok, sub * 4 + e)] = f2e4m3(u[e]);
        blk8[vswz8_off(tok, 64 + sub * 4 + e)] = f2e4m3(w[e]);
      } else {
        blk[vswz_off(tok, sub * 4 + e)] = f2bf(u[e]);
        blk[vswz_off(tok, 64 + sub * 4 + e)] = f2bf(w[e]);
      }
    }
    return;
  }
  if (a.qk_norm) {
    const float inv = 1.0f / sqrtf(ss / 128.0f + a.eps);
    const float gl[4] = {bf2f((bf16_t)(glo.x & 0xffff)), bf2f((bf16_t)(glo.x >> 16)),
                         bf2f((bf16_t)(glo.y & 0xffff)), bf2f((bf16_t)(glo.y >> 16))};
    const float gh[4] = {bf2f((bf16_t)(ghi.x & 0xffff)), bf2f((bf16_t)(ghi.x >> 16)),
                         bf2f((bf16_t)(ghi.y & 0xffff)), bf2f((bf16_t)(ghi.y >> 16))};
#pragma unroll
    for (int e = 0; e < 4; e++) { u[e] = u[e] * inv * gl[e]; w[e] = w[e] * inv * gh[e]; }
  }
  const float c[4] = {cs0.x, cs0.z, cs1.x, cs1.z}, sn[4] = {cs0.y, cs0.w, cs1.y, cs1.w};
  float r1[4], r2[4];
#pragma unroll
  for (int e = 0; e < 4; e++) {
    r1[e] = __builtin_fmaf(u[e], c[e], -(w[e] * sn[e]));
    r2[e] = __builtin_fmaf(w[e], c[e], u[e] * sn[e]);
  }
  if constexpr (FP8) {
    if (!is_q) {   // 4 consecutive dims = 4 consecutive bytes of one lane slot
      *(uint32_t*)(blk8 + kswz8_off(tok, sub * 4)) = f2e4m3x4(r1[0], r1[1], r1[2], r1[3]);
      *(uint32_t*)(blk8 + kswz8_off(tok, 64 + sub * 4)) = f2e4m3x4(r2[0], r2[1], r2[2], r2[3]);
      return;
    }
  }
  *w1 = make_uint2((uint32_t)f2bf(r1[0]) | ((uint32_t)f2bf(r1[1]) << 16), (uint32_t)f2bf(r1[2]) | ((uint32_t)f2bf(r1[3]) << 16));
  *w2 = make_uint2((uint32_t)f2bf(r2[0]) | ((uint32_t)f2bf(r2[1]) << 16), (uint32_t)f2bf(r2[2]) | ((uint32_t)f2bf(r2[3]) << 16));
  if (!is_q) {   // 4 consecutive dims lie in one 8-element lane slot of the swizzled key block
    *(uint2*)(blk + kswz_off(tok, sub * 4)) = *w1;
    *(uint2*)(blk + kswz_off(tok, 64 + sub * 4)) = *w2;
  }
}
