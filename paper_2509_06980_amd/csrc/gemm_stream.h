// Weight-streaming GEMM for decode batches (up to 128 rows): C[M,N] = A[M,K] * W[N,K]^T.
#pragma once
#include "kernels.h"

typedef __amdgpu_buffer_rsrc_t buf_rsrc;
__device__ __forceinline__ u32x4 buf_load(buf_rsrc r, int voff, int soff) {
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}

template <int EPI, int RB, int CB, int D>
__global__ __launch_bounds__(256) void gemm_stream_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ Wp,
                                                          void* __restrict__ Cv, int M, int N, int K, int splits,
                                                          int steps_per_split, float* __restrict__ zt) {
  constexpr int UNITS = RB * CB;
  constexpr int OWN = (UNITS + 3) / 4;          // units a wave finishes: [wave * OWN, ...)
  extern __shared__ f32x4 red[];                // [unit][3][64]
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int tile = blockIdx.x / splits, split = blockIdx.x - tile * splits;
  const int nsteps = K >> 5, NB = N >> 5, N16 = N >> 4;
  const int t0 = split * steps_per_split, t1 = min(t0 + steps_per_split, nsteps);
  const int lw = ((lane >> 5) << 10) + (((lane & 15) + (((lane >> 4) & 1) << 5)) << 4);
  const int la = ((lane >> 5) << 12) + (((lane & 15) + (((lane >> 4) & 1) << 5)) << 4);
  const buf_rsrc ra = __builtin_amdgcn_make_buffer_rsrc((void*)A, 0, K * 256, 0x00027000);
  const buf_rsrc rw = __builtin_amdgcn_make_buffer_rsrc((void*)Wp, 0, (unsigned)N * K * 2u, 0x00027000);
  unsigned wcol[CB];
#pragma unroll
  for (int c = 0; c < CB; c++) {
    const int c16 = min(tile * CB + c, N16 - 1);
    wcol[c] = (unsigned)(c16 >> 1) * 4096u + (c16 & 1) * 256u;
  }
  f32x4 acc[CB][RB];
#pragma unroll
  for (int c = 0; c < CB; c++)
#pragma unroll
    for (int r = 0; r < RB; r++) acc[c][r] = (f32x4){0.f, 0.f, 0.f, 0.f};
  u32x4 w[D][CB], a[D][RB];
#define GS_LOAD(S, T)                                                                        \
  {                                                                                          \
    const int t_ = (T);                                                                      \
    const bool in_ = t_ < t1;                                                                \
    const unsigned ws_ = (unsigned)(t_ >> 1) * (unsigned)NB * 4096u + (t_ & 1) * 2048u;      \
    const int vw_ = in_ ? lw : 0x7fff0000, va_ = in_ ? la : 0x7fff0000;                      \
    _Pragma("unroll") for (int c = 0; c < CB; c++) w[S][c] = buf_load(rw, vw_, in_ ? ws_ + wcol[c] : 0); \
    _Pragma("unroll") for (int r = 0; r < RB; r++)                                           \
      a[S][r] = buf_load(ra, va_ + (r >> 1) * 1024 + (r & 1) * 256, in_ ? t_ * 8192 : 0);    \
    __builtin_amdgcn_sched_barrier(0);                                                       \
  }
#pragma unroll
  for (int d = 0; d < D; d++) GS_LOAD(d, t0 + wave + 4 * d)
  for (int t = t0 + wave; t < t1; t += 4 * D) {
#pragma unroll
    for (int d = 0; d < D; d++) {
      if (t + 4 * d < t1) {
#pragma unroll
        for (int c = 0; c < CB; c++)
#pragma unroll
          for (int r = 0; r < RB; r++)
            acc[c][r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[d][c]),
                                                                __builtin_bit_cast(bf16x8, a[d][r]), acc[c][r], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      GS_LOAD(d, t + 4 * (d + D))
    }
  }
#undef GS_LOAD
  // unit u = r * CB + c; wave v of the other three: slot (v - owner - 1) & 3
#pragma unroll
  for (int r = 0; r < RB; r++)
#pragma unroll
    for (int c = 0; c < CB; c++) {
      const int u = r * CB + c, owner = u / OWN;
      if (owner != wave) red[(u * 3 + ((wave - owner - 1) & 3)) * 64 + lane] = acc[c][r];
    }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < RB; r++)
#pragma unroll
    for (int c = 0; c < CB; c++) {
      const int u = r * CB + c, owner = u / OWN;
      if (owner != wave) continue;
      f32x4 v = acc[c][r];
#pragma unroll
      for (int x = 0; x < 3; x++) v += red[(u * 3 + x) * 64 + lane];
      const int row = r * 16 + (lane & 15), c16 = tile * CB + c;
      if (c16 >= N16) continue;
      if (EPI == EPI_SWIGLU) {
        f32x4 up;
#pragma unroll
        for (int i = 0; i < 4; i++) up[i] = __shfl_xor(v[i], 32, 64);
        if (lane < 32 && row < M) {
          uint32_t y[4];
#pragma unroll
          for (int i = 0; i < 4; i++) y[i] = f2bf(v[i] / (1.0f + __expf(-v[i])) * up[i]);
          *(uint2*)((bf16_t*)Cv + atile_off(row, c16 * 8 + 4 * (lane >> 4), N >> 1)) =
              make_uint2(y[0] | (y[1] << 16), y[2] | (y[3] << 16));
        }
      } else if (row < M) {
        float* C = (float*)Cv + (size_t)split * M * N;
        __builtin_nontemporal_store(v, (f32x4*)(C + (size_t)row * N + c16 * 16 + 4 * (lane >> 4)));
      }
    }
}
