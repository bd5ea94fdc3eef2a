// Shape-generic kernels: fp32 mode, and bf16 models whose shape the MFMA kernels do not cover.
// One decoder block of the policy pi_theta(a | s_t) (paper Section 2.2) is
//   h += W_o attn(rope(norm(W_q a)), rope(norm(W_k a)), W_v a),  a = rmsnorm(h)
//   h += W_down (silu(W_gate b) * W_up b),                       b = rmsnorm(h)
// Each kernel below is one of those pieces; accumulation is always fp32.
#include "kernels.h"
#include "qkrope.h"

template <typename TW>
__global__ void embed_kernel(const TW* __restrict__ E, const int32_t* __restrict__ tok,
                             float* __restrict__ h, int H) {
  int row = blockIdx.x;
  const TW* e = E + (size_t)tok[row] * H;
  for (int j = threadIdx.x; j < H; j += blockDim.x) h[(size_t)row * H + j] = ldf(e + j);
}

template <typename TW, typename TA>
__global__ void rmsnorm_kernel(const float* __restrict__ h, const TW* __restrict__ g,
                               TA* __restrict__ out, int H, float eps) {
  __shared__ float red[4];
  int row = blockIdx.x;
  const float* x = h + (size_t)row * H;
  float ss = 0.f;
  for (int j = threadIdx.x; j < H; j += 256) ss += x[j] * x[j];
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  float tot = red[0] + red[1] + red[2] + red[3];
  float inv = 1.0f / sqrtf(tot / (float)H + eps);
  for (int j = threadIdx.x; j < H; j += 256) stf(out + (size_t)row * H + j, x[j] * inv * ldf(g + j));
}

// grid M, block 256: h[row] += sum_p parts[p][row]; out = rmsnorm(h[row]) * g, A-tile layout
__global__ void add_rmsnorm_kernel(float* __restrict__ h, const float* __restrict__ parts, int n_part,
                                   size_t part_stride, const bf16_t* __restrict__ g,
                                   bf16_t* __restrict__ out, int H, float eps,
                                   const int32_t* __restrict__ rows) {
  __shared__ float red[4];
  const int orow = blockIdx.x;
  const int row = rows ? rows[orow] : orow;
  float* x = h + (size_t)row * H;
  const float* pr = parts + (size_t)row * H;
  float ss = 0.f;
  for (int j = threadIdx.x * 4; j < H; j += 1024) {
    float4 v = *(const float4*)(x + j);
    int p = 0;
    for (; p + 4 <= n_part; p += 4) {     // four independent loads in flight, added in order
      float4 u0 = *(const float4*)(pr + (size_t)p * part_stride + j);
      float4 u1 = *(const float4*)(pr + (size_t)(p + 1) * part_stride + j);
      float4 u2 = *(const float4*)(pr + (size_t)(p + 2) * part_stride + j);
      float4 u3 = *(const float4*)(pr + (size_t)(p + 3) * part_stride + j);
      v.x = (((v.x + u0.x) + u1.x) + u2.x) + u3.x;
      v.y = (((v.y + u0.y) + u1.y) + u2.y) + u3.y;
      v.z = (((v.z + u0.z) + u1.z) + u2.z) + u3.z;
      v.w = (((v.w + u0.w) + u1.w) + u2.w) + u3.w;
    }
    for (; p < n_part; p++) {
      float4 u = *(const float4*)(pr + (size_t)p * part_stride + j);
      v.x += u.x; v.y += u.y; v.z += u.z; v.w += u.w;
    }
    if (n_part > 0) *(float4*)(x + j) = v;
    ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
  }
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();   // also makes every thread's updated h visible to the block
  float inv = 1.0f / sqrtf((red[0] + red[1] + red[2] + red[3]) / (float)H + eps);
  for (int j = threadIdx.x * 8; j < H; j += 2048) {
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; e++) {
      float y0 = x[j + 2 * e] * inv * bf2f(g[j + 2 * e]);
      float y1 = x[j + 2 * e + 1] * inv * bf2f(g[j + 2 * e + 1]);
      w[e] = (uint32_t)f2bf(y0) | ((uint32_t)f2bf(y1) << 16);
    }
    *(uint4*)(out + atile_off(orow, j, H)) = make_uint4(w[0], w[1], w[2], w[3]);
  }
}

// Same operation with the whole row in registers: every load of the row and of its (up to NP)
// partial sums is issued before the first use, so a row costs about one memory round trip instead
// of one per group of partials; the normalised row is written from registers.  H <= ITER * 1024.
// A row's output is 16-byte pieces 512 bytes apart (operand layout); 8 consecutive rows fill a 128-byte
// line.  Workgroups are handed to the 8 XCDs round-robin, so 8 consecutive rows are given to workgroups
// of one XCD, whose L2 then writes whole lines: H = 2560, 8192 rows, one partial sum 72 -> 56 us (5.2 TB/s),
// none 41 -> 25 us, 587 rows with five 12.9 -> 11.0 us.  Below 256 rows the launch is one latency chain
// and rows stay in launch order (128 rows with two partial sums 5.4 against 6.0 us).
// EMB: the row is the embedding of token tok[row] instead, written to h on the way (first norm of a pass):
// one launch and one reading of h less (8192 x 2560: 36 + 25 -> 43 us, 6 x 4096: 9.3 + 3.6 -> 4.7 us).
template <int ITER, int NP, bool EMB>
__global__ __launch_bounds__(256) void add_rmsnorm_reg_kernel(
    float* __restrict__ h, const float* __restrict__ parts, int n_part, size_t part_stride,
    const bf16_t* __restrict__ g, bf16_t* __restrict__ out, int H, float eps,
    const int32_t* __restrict__ rows, int M, const bf16_t* __restrict__ embed, const int32_t* __restrict__ tok) {
  __shared__ float red[4];
  const int id = blockIdx.x;
  const int orow = M < 256 ? id : (id & ~63) + (id & 7) * 8 + (id >> 3 & 7);
  if (orow >= M) return;
  const int row = rows ? rows[orow] : orow;
  float* x = h + (size_t)row * H;
  const float* pr = parts + (size_t)row * H;
  const bf16_t* e = EMB ? embed + (size_t)tok[row] * H : nullptr;
  float4 v[ITER], u[ITER][NP];
  uint2 gw[ITER];
#pragma unroll
  for (int it = 0; it < ITER; it++) {
    const int j = threadIdx.x * 4 + it * 1024;
    const bool ok = j < H;
    gw[it] = ok ? *(const uint2*)(g + j) : make_uint2(0u, 0u);
    if constexpr (EMB) {
      const uint2 w = ok ? *(const uint2*)(e + j) : make_uint2(0u, 0u);
      v[it] = make_float4(bf2f((bf16_t)(w.x & 0xffff)), bf2f((bf16_t)(w.x >> 16)),
                          bf2f((bf16_t)(w.y & 0xffff)), bf2f((bf16_t)(w.y >> 16)));
      continue;
    }
    v[it] = ok ? *(const float4*)(x + j) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int p = 0; p < NP; p++)
      u[it][p] = (ok && p < n_part) ? *(const float4*)(pr + (size_t)p * part_stride + j)
                                    : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  float ss = 0.f;
#pragma unroll
  for (int it = 0; it < ITER; it++) {
#pragma unroll
    for (int p = 0; p < NP; p++)
      if (!EMB && p < n_part) {   // ascending order, as the looping kernel adds them
        v[it].x += u[it][p].x; v[it].y += u[it][p].y; v[it].z += u[it][p].z; v[it].w += u[it][p].w;
      }
    const int j = threadIdx.x * 4 + it * 1024;
    if ((EMB || n_part > 0) && j < H) *(float4*)(x + j) = v[it];
    ss += v[it].x * v[it].x + v[it].y * v[it].y + v[it].z * v[it].z + v[it].w * v[it].w;
  }
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  const float inv = 1.0f / sqrtf((red[0] + red[1] + red[2] + red[3]) / (float)H + eps);
#pragma unroll
  for (int it = 0; it < ITER; it++) {
    const int j = threadIdx.x * 4 + it * 1024;
    if (j < H) {
      float y0 = v[it].x * inv * bf2f((bf16_t)(gw[it].x & 0xffff));
      float y1 = v[it].y * inv * bf2f((bf16_t)(gw[it].x >> 16));
      float y2 = v[it].z * inv * bf2f((bf16_t)(gw[it].y & 0xffff));
      float y3 = v[it].w * inv * bf2f((bf16_t)(gw[it].y >> 16));
      uint2 w;
      w.x = (uint32_t)f2bf(y0) | ((uint32_t)f2bf(y1) << 16);
      w.y = (uint32_t)f2bf(y2) | ((uint32_t)f2bf(y3) << 16);
      *(uint2*)(out + atile_off(orow, j, H)) = w;   // 4 consecutive k share one 16-byte lane slot
    }
  }
}

template <int NP, bool EMB>
static void launch_add_rmsnorm_reg(hipStream_t s, float* h, const float* parts, int n_part, size_t part_stride,
                                   const bf16_t* g, bf16_t* out, int M, int H, float eps, const int32_t* rows,
                                   const bf16_t* embed, const int32_t* tok) {
  const int grid = M < 256 ? M : (M + 63) / 64 * 64;
  auto go = [&](auto kernel) {
    kernel<<<grid, 256, 0, s>>>(h, parts, n_part, part_stride, g, out, H, eps, rows, M, embed, tok);
  };
  if (H <= 1024) go(add_rmsnorm_reg_kernel<1, NP, EMB>);
  else if (H <= 2048) go(add_rmsnorm_reg_kernel<2, NP, EMB>);
  else if (H <= 3072) go(add_rmsnorm_reg_kernel<3, NP, EMB>);
  else go(add_rmsnorm_reg_kernel<4, NP, EMB>);
}

void launch_add_rmsnorm(hipStream_t s, float* h, const float* parts, int n_part, size_t part_stride,
                        const bf16_t* g, bf16_t* out, int M, int H, float eps, const int32_t* rows) {
  if (M <= 0) return;
  if (n_part <= 8 && H % 4 == 0 && H <= 4096) {
    // registers for one partial sum only where there is no more: 8 blocks instead of 3 share a CU
    if (n_part <= 1) launch_add_rmsnorm_reg<1, false>(s, h, parts, n_part, part_stride, g, out, M, H, eps, rows, nullptr, nullptr);
    else launch_add_rmsnorm_reg<8, false>(s, h, parts, n_part, part_stride, g, out, M, H, eps, rows, nullptr, nullptr);
    return;
  }
  add_rmsnorm_kernel<<<M, 256, 0, s>>>(h, parts, n_part, part_stride, g, out, H, eps, rows);
}

void launch_embed_rmsnorm(hipStream_t s, const bf16_t* embed, const int32_t* tok, float* h, const bf16_t* g,
                          bf16_t* out, int M, int H, float eps) {
  if (M <= 0) return;
  if (H % 4 == 0 && H <= 4096) {
    launch_add_rmsnorm_reg<1, true>(s, h, nullptr, 0, 0, g, out, M, H, eps, nullptr, embed, tok);
    return;
  }
  launch_embed<bf16_t>(s, embed, tok, h, M, H);
  launch_add_rmsnorm(s, h, nullptr, 0, 0, g, out, M, H, eps, nullptr);
}

template <typename TA, typename TW>
__global__ __launch_bounds__(256) void gemm_generic_kernel(const TA* __restrict__ A,
                                                           const TW* __restrict__ W,
                                                           float* __restrict__ C, int M, int N,
                                                           int K, int accumulate) {
  __shared__ float As[16][65];
  __shared__ float Ws[16][65];
  int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  int tid = threadIdx.x, ty = tid >> 4, tx = tid & 15;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < K; k0 += 16) {
#pragma unroll
    for (int i = 0; i < 4; i++) {
      int e = tid + i * 256, r = e >> 4, kk = e & 15;
      int gm = m0 + r, gn = n0 + r, gk = k0 + kk;
      As[kk][r] = (gm < M && gk < K) ? ldf(A + (size_t)gm * K + gk) : 0.f;
      Ws[kk][r] = (gn < N && gk < K) ? ldf(W + (size_t)gn * K + gk) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; kk++) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; i++) { a[i] = As[kk][ty * 4 + i]; b[i] = Ws[kk][tx * 4 + i]; }
#pragma unroll
      for (int i = 0; i < 4; i++)
#pragma unroll
        for (int j = 0; j < 4; j++) acc[i][j] += a[i] * b[j];
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; i++)
#pragma unroll
    for (int j = 0; j < 4; j++) {
      int gm = m0 + ty * 4 + i, gn = n0 + tx * 4 + j;
      if (gm < M && gn < N) {
        float* c = C + (size_t)gm * N + gn;
        *c = accumulate ? *c + acc[i][j] : acc[i][j];
      }
    }
}

// The same product on the fp32 matrix instruction (16x16x4: exact fp32 products, fp32 accumulation), for
// rows of whole 4-element pieces.  A wave forms 16 R rows x 16 columns with no LDS in its loop: lane
// (i = lane % 16, g = lane / 16) reads four consecutive k of row (column) i at k0 + 4 g and feeds
// component c of both operands to MFMA c, whose k index is then k0 + 4 g + c on either side.  The eight
// waves of a workgroup take every eighth 16-k step, several steps in flight, and the eight sums are added in ascending
// order, a row of each group of four per wave.  At the few rows of a decode step a launch is
// a chain of memory round trips, not arithmetic: K / 768 of them here, against K / 16 with two barriers
// each in the tile kernel above, which keeps the shapes whose rows are not whole pieces (4 rows: K = 256
// 30 -> 2.7 us, K = 688 85 -> 4.5 us, 5.6 with four waves; 51 200 rows at hidden 1024, fp32: a two-layer prefill 138 -> 95 ms
// with four waves, 82 ms with eight and the norm inside).
constexpr int kWaves32 = 8;
template <typename TA, typename TW, int R>
__global__ __launch_bounds__(64 * kWaves32) void gemm_mfma32_kernel(const TA* __restrict__ A, const TW* __restrict__ W,
                                                          float* __restrict__ C, int M, int N, int K,
                                                          int accumulate) {
  __shared__ f32x4 red[R][kWaves32][64];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, i = lane & 15, g = lane >> 4;
  const int n0 = blockIdx.x * 16, m0 = blockIdx.y * (16 * R);
  const TW* w = W + (size_t)min(n0 + i, N - 1) * K;      // rows and columns past the end: repeated, not stored
  const TA* a[R];
#pragma unroll
  for (int r = 0; r < R; r++) a[r] = A + (size_t)min(m0 + 16 * r + i, M - 1) * K;
  f32x4 acc[R];
#pragma unroll
  for (int r = 0; r < R; r++) acc[r] = (f32x4){0.f, 0.f, 0.f, 0.f};
  constexpr int U = R == 1 ? 6 : 2, STEP = 16 * kWaves32;   // 16-k steps in flight
  for (int k0 = wave * 16; k0 < K; k0 += STEP * U) {
    float wv[U][4], av[U][R][4];
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int k = k0 + STEP * u + 4 * g;
      const bool in = k < K;                             // K % 4 == 0: a piece is inside or outside as a whole
#pragma unroll
      for (int e = 0; e < 4; e++) wv[u][e] = 0.f;
      if (in) ld4(w + k, wv[u][0], wv[u][1], wv[u][2], wv[u][3]);
#pragma unroll
      for (int r = 0; r < R; r++) {
#pragma unroll
        for (int e = 0; e < 4; e++) av[u][r][e] = 0.f;
        if (in) ld4(a[r] + k, av[u][r][0], av[u][r][1], av[u][r][2], av[u][r][3]);
      }
    }
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
      for (int e = 0; e < 4; e++)
#pragma unroll
        for (int r = 0; r < R; r++)
          acc[r] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u][r][e], wv[u][e], acc[r], 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < R; r++) red[r][wave][lane] = acc[r];
  __syncthreads();
  const int n = n0 + i;
  if (n >= N) return;
#pragma unroll
  for (int x = 0; x < 4 * R; x += kWaves32) {      // one row of every four-row group of a block per wave
    const int y = x + wave, r = y >> 2, e = y & 3;
    if (y >= 4 * R) break;
    // the same order for every row: a row's bits do not depend on where it lies in the batch
    float v = red[r][0][lane][e];
#pragma unroll
    for (int q = 1; q < kWaves32; q++) v += red[r][q][lane][e];
    const int row = m0 + 16 * r + 4 * g + e;
    if (row < M) {
      float* c = C + (size_t)row * N + n;
      *c = accumulate ? *c + v : v;
    }
  }
}

// fp32 models: rmsnorm and the product behind it in one launch, C[M, N] = (rmsnorm(h) g) W^T, and with SWIGLU also the
// activation: W holds N gate rows, then N up rows, C = silu(gate) * up.  The loop of gemm_mfma32_kernel; the rows of h pass
// through every workgroup anyway, so each sums their squares on the way and divides its 16 columns at the end (the factor
// of a row commutes with the product).  A pass of a few rows is a chain of launches of 2 to 5 us; this takes out the norms (2.0 us
// each and the gap) and the activation (2.3 us): gate-up at 4 rows, K = 256, N = 688 2.0 + 3.3 + 2.3 -> 4.7 us.  EMB: the rows are the embeddings of tok, written to h by the first
// column of workgroups.
template <int R, bool SWIGLU, bool EMB>
__global__ __launch_bounds__(64 * kWaves32) void norm_gemm32_kernel(float* h, const float* __restrict__ E,
                                                          const int32_t* __restrict__ tok, const float* __restrict__ gain,
                                                          const float* __restrict__ W, float* __restrict__ C, int M, int N,
                                                          int K, float eps) {
  constexpr int S = SWIGLU ? 2 : 1;
  __shared__ f32x4 red[S][R][kWaves32][64];
  __shared__ float sq[R][kWaves32][16];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, i = lane & 15, g = lane >> 4;
  const int n0 = blockIdx.x * 16, m0 = blockIdx.y * (16 * R), n = n0 + i;
  const float* w[S];
#pragma unroll
  for (int s = 0; s < S; s++) w[s] = W + ((size_t)s * N + min(n, N - 1)) * K;    // rows and columns past the end: repeated, not stored
  const float* a[R];
#pragma unroll
  for (int r = 0; r < R; r++) {
    const int row = min(m0 + 16 * r + i, M - 1);
    a[r] = EMB ? E + (size_t)tok[row] * K : h + (size_t)row * K;
  }
  f32x4 acc[S][R];
  float ss[R];
#pragma unroll
  for (int r = 0; r < R; r++) {
    ss[r] = 0.f;
#pragma unroll
    for (int s = 0; s < S; s++) acc[s][r] = (f32x4){0.f, 0.f, 0.f, 0.f};
  }
  constexpr int U = R == 1 ? 4 : 2, STEP = 16 * kWaves32;
  for (int k0 = wave * 16; k0 < K; k0 += STEP * U) {
    float wv[U][S][4], av[U][R][4], gv[U][4];
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int k = k0 + STEP * u + 4 * g;
      const bool in = k < K;                             // K % 4 == 0: a piece is inside or outside as a whole
      const float zero = 0.f;
      auto get = [&](const float* p, float (&x)[4]) {
        x[0] = x[1] = x[2] = x[3] = zero;
        if (in) ld4(p + k, x[0], x[1], x[2], x[3]);
      };
      get(gain, gv[u]);
#pragma unroll
      for (int s = 0; s < S; s++) get(w[s], wv[u][s]);
#pragma unroll
      for (int r = 0; r < R; r++) {
        get(a[r], av[u][r]);
        if (EMB && in && blockIdx.x == 0 && m0 + 16 * r + i < M)
          *(f32x4*)(h + (size_t)(m0 + 16 * r + i) * K + k) = (f32x4){av[u][r][0], av[u][r][1], av[u][r][2], av[u][r][3]};
      }
    }
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
      for (int e = 0; e < 4; e++)
#pragma unroll
        for (int r = 0; r < R; r++) {
          ss[r] = __builtin_fmaf(av[u][r][e], av[u][r][e], ss[r]);
          const float x = av[u][r][e] * gv[u][e];
#pragma unroll
          for (int s = 0; s < S; s++) acc[s][r] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, wv[u][s][e], acc[s][r], 0, 0, 0);
        }
  }
#pragma unroll
  for (int r = 0; r < R; r++) {
#pragma unroll
    for (int s = 0; s < S; s++) red[s][r][wave][lane] = acc[s][r];
    ss[r] += __shfl_xor(ss[r], 16, 64);
    ss[r] += __shfl_xor(ss[r], 32, 64);
    if (lane < 16) sq[r][wave][lane] = ss[r];
  }
  __syncthreads();
  if (n >= N) return;
#pragma unroll
  for (int x = 0; x < 4 * R; x += kWaves32) {      // one row of every four-row group of a block per wave
    const int y = x + wave, r = y >> 2, e = y & 3, m = 4 * g + e, row = m0 + 16 * r + m;
    if (y >= 4 * R) break;
    // the same order for every row: a row's bits do not depend on where it lies in the batch
    float v[S], t = sq[r][0][m];
#pragma unroll
    for (int s = 0; s < S; s++) v[s] = red[s][r][0][lane][e];
#pragma unroll
    for (int q = 1; q < kWaves32; q++) {
      t += sq[r][q][m];
#pragma unroll
      for (int s = 0; s < S; s++) v[s] += red[s][r][q][lane][e];
    }
    if (row >= M) continue;
    const float inv = 1.0f / sqrtf(t / (float)K + eps);
    float z = v[0] * inv;
    if (SWIGLU) z = z / (1.0f + expf(-z)) * (v[S - 1] * inv);
    C[(size_t)row * N + n] = z;
  }
}

// fp32 models, few rows: rmsnorm, one head's QKV projection, QK-norm, RoPE and the cache write in one launch (grid: heads x blocks
// of 16 rows).  D: head_dim, 64 or 128.  The waves share K as above; the head's 16 x D block is put together in LDS,
// where 32 lanes then own a row's head.  Against the product and the norm / RoPE kernel: two launches and the fp32 projection
// less (4 rows, 8 heads of 64, K = 256: 2.0 + 3.4 + 3.2 -> 6.0 us and two gaps); but a head is one workgroup's, which
// reads D K weights alone, so it is for small K (see the launcher).
template <int D, bool EMB>
__global__ __launch_bounds__(64 * kWaves32) void norm_qkv32_kernel(float* h, const float* __restrict__ E, const int32_t* __restrict__ tok,
                                                         const float* __restrict__ gain, const float* __restrict__ W,
                                                         const float* __restrict__ gq, const float* __restrict__ gk,
                                                         const float* __restrict__ rope_cs, const int32_t* __restrict__ row_pos,
                                                         const int32_t* __restrict__ row_slot,
                                                         const int32_t* __restrict__ page_table, float* __restrict__ qout,
                                                         float* __restrict__ kpool, float* __restrict__ vpool, int nq, int nkv,
                                                         int M, int K, float eps, int qk_norm, int pt_stride) {
  constexpr int CB = D / 16, U = 2, HALF = D / 2, LPR = 4 * kWaves32, PP = HALF / LPR, STEP = 16 * kWaves32;
  __shared__ f32x4 red[kWaves32][CB][64];
  __shared__ float xs[16][D + 1], sq[kWaves32][16];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, i = lane & 15, g = lane >> 4;
  const int hd = blockIdx.x, m0 = blockIdx.y * 16;
  const float* w = W + ((size_t)hd * D + i) * K;
  const int arow = min(m0 + i, M - 1);
  const float* a = EMB ? E + (size_t)tok[arow] * K : h + (size_t)arow * K;
  // what the end needs, asked for first: LPR lanes own a row's head, each PP pairs of dims
  const int x = tid / LPR, sub = tid % LPR, row = m0 + x, prow = min(row, M - 1);
  const bool is_q = hd < nq, is_v = hd >= nq + nkv;
  const int pos = row_pos[prow], page = page_table[(size_t)row_slot[prow] * pt_stride + (pos >> 4)];
  float cs[PP], sn[PP], g1[PP], g2[PP];
#pragma unroll
  for (int j = 0; j < PP; j++) {
    const int d = sub + LPR * j;
    cs[j] = rope_cs[((size_t)pos * HALF + d) * 2];
    sn[j] = rope_cs[((size_t)pos * HALF + d) * 2 + 1];
    g1[j] = (is_q ? gq : gk)[d];
    g2[j] = (is_q ? gq : gk)[d + HALF];
  }
  f32x4 acc[CB];
#pragma unroll
  for (int c = 0; c < CB; c++) acc[c] = (f32x4){0.f, 0.f, 0.f, 0.f};
  float ss = 0.f;
  for (int k0 = wave * 16; k0 < K; k0 += STEP * U) {
    float wv[U][CB][4], av[U][4], gv[U][4];
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int k = k0 + STEP * u + 4 * g;
      const bool in = k < K;
      auto get = [&](const float* p, float (&x)[4]) {
        x[0] = x[1] = x[2] = x[3] = 0.f;
        if (in) ld4(p + k, x[0], x[1], x[2], x[3]);
      };
      get(a, av[u]);
      get(gain, gv[u]);
#pragma unroll
      for (int c = 0; c < CB; c++) get(w + (size_t)c * 16 * K, wv[u][c]);
      if (EMB && in && hd == 0 && m0 + i < M)
        *(f32x4*)(h + (size_t)(m0 + i) * K + k) = (f32x4){av[u][0], av[u][1], av[u][2], av[u][3]};
    }
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
      for (int e = 0; e < 4; e++) {
        ss = __builtin_fmaf(av[u][e], av[u][e], ss);
        const float x = av[u][e] * gv[u][e];
#pragma unroll
        for (int c = 0; c < CB; c++) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, wv[u][c][e], acc[c], 0, 0, 0);
      }
  }
#pragma unroll
  for (int c = 0; c < CB; c++) red[wave][c][lane] = acc[c];
  ss += __shfl_xor(ss, 16, 64);
  ss += __shfl_xor(ss, 32, 64);
  if (lane < 16) sq[wave][lane] = ss;
  __syncthreads();
  if (wave < CB) {
    f32x4 v = red[0][wave][lane];
#pragma unroll
    for (int q = 1; q < kWaves32; q++) v += red[q][wave][lane];
#pragma unroll
    for (int e = 0; e < 4; e++) xs[4 * g + e][16 * wave + i] = v[e];
  }
  __syncthreads();
  if (row >= M) return;          // whole groups of LPR lanes; no barrier below
  float t = sq[0][x];
#pragma unroll
  for (int q = 1; q < kWaves32; q++) t += sq[q][x];
  const float inv_row = 1.0f / sqrtf(t / (float)K + eps);
  float lo[PP], hi[PP], s2 = 0.f;
#pragma unroll
  for (int j = 0; j < PP; j++) {
    lo[j] = xs[x][sub + LPR * j] * inv_row;
    hi[j] = xs[x][sub + LPR * j + HALF] * inv_row;
    s2 = __builtin_fmaf(hi[j], hi[j], __builtin_fmaf(lo[j], lo[j], s2));
  }
#pragma unroll
  for (int o = LPR / 2; o > 0; o >>= 1) s2 += __shfl_xor(s2, o, LPR);
  const float inv = (qk_norm && !is_v) ? 1.0f / sqrtf(s2 / (float)D + eps) : 1.0f;
  float* dst = is_q ? qout + ((size_t)row * nq + hd) * D
                    : (is_v ? vpool : kpool) + (((size_t)page * nkv + (is_v ? hd - nq - nkv : hd - nq)) * RL_PAGE + (pos & (RL_PAGE - 1))) * D;
#pragma unroll
  for (int j = 0; j < PP; j++) {
    const int d = sub + LPR * j;
    float u = lo[j], v = hi[j];
    if (!is_v) {
      if (qk_norm) { u = u * inv * g1[j]; v = v * inv * g2[j]; }
      const float y = u * cs[j] - v * sn[j];
      v = v * cs[j] + u * sn[j];
      u = y;
    }
    dst[d] = u;
    dst[d + HALF] = v;
  }
}

// grid (M, nq + 2 nkv), block 64
template <typename TW, typename TA, typename TKV>
__global__ void qkrope_kernel(const float* __restrict__ qkv, const TW* __restrict__ gq,
                              const TW* __restrict__ gk, const float* __restrict__ rope_cs,
                              const int32_t* __restrict__ row_pos,
                              const int32_t* __restrict__ row_slot,
                              const int32_t* __restrict__ page_table, TA* __restrict__ qout,
                              TKV* __restrict__ kpool, TKV* __restrict__ vpool, int nq, int nkv,
                              int d, float eps, int qk_norm, int pt_stride) {
  int row = blockIdx.x, hd = blockIdx.y, half = d >> 1;
  int pos = row_pos[row];
  const float* x = qkv + (size_t)row * (nq + 2 * nkv) * d + (size_t)hd * d;
  bool is_q = hd < nq, is_v = hd >= nq + nkv;
  float x1[2], x2[2];
  float ss = 0.f;
  int cnt = 0;
  for (int i = threadIdx.x; i < half; i += 64, cnt++) {
    const float u = x[i], w = x[i + half];
    x1[cnt] = u;
    x2[cnt] = w;
    ss += __builtin_fmaf(w, w, u * u);
  }
  ss = wave_sum(ss);
  float inv = (qk_norm && !is_v) ? 1.0f / sqrtf(ss / (float)d + eps) : 1.0f;
  TKV* blk = nullptr;
  int tok = pos & (RL_PAGE - 1);
  if (!is_q) {
    int page = page_table[(size_t)row_slot[row] * pt_stride + (pos >> 4)];
    int kvh = is_v ? hd - nq - nkv : hd - nq;
    blk = (is_v ? vpool : kpool) + ((size_t)page * nkv + kvh) * (RL_PAGE * d);
  }
  const TW* g = is_q ? gq : gk;
  cnt = 0;
  for (int i = threadIdx.x; i < half; i += 64, cnt++) {
    float a = x1[cnt], b = x2[cnt];
    if (is_v) {
      stf(blk + tok * d + i, a);
      stf(blk + tok * d + i + half, b);
      continue;
    }
    if (qk_norm) { a = a * inv * ldf(g + i); b = b * inv * ldf(g + i + half); }
    float c = rope_cs[((size_t)pos * half + i) * 2], s = rope_cs[((size_t)pos * half + i) * 2 + 1];
    float y1 = a * c - b * s, y2 = b * c + a * s;
    if (is_q) {
      stf(qout + (size_t)row * nq * d + (size_t)hd * d + i, y1);
      stf(qout + (size_t)row * nq * d + (size_t)hd * d + i + half, y2);
    } else {
      stf(blk + tok * d + i, y1);
      stf(blk + tok * d + i + half, y2);
    }
  }
}

// grid (M, nq), block 256: one workgroup per (row, q head).  Sixteen groups of 16 lanes: group g takes
// the tokens at offset g of every page, lane `sub` of it holds a sixteenth of the head (VEC, head_dim a
// multiple of 4: dims 64 j + 4 sub .. + 3, one 16-byte read each in fp32; else dims 16 j + sub), so that
// a wave reads whole rows.  Four pages' page ids, keys and values are requested before the first use;
// every group keeps an online softmax of its own and the sixteen are joined through LDS.  A chain of
// one memory round trip per 64 tokens (4 rows x 4 heads at 32 to 104 tokens: 13.7 -> 5.0 us; 64 rows at 800
// tokens, head_dim 64: a decode step of 2 layers 1200 -> 202 us together with the product above; one
// wave had read a token's dims one after the other).
template <typename TA, typename TKV, bool VEC>
__global__ __launch_bounds__(256) void attention_generic_kernel(
    const TA* __restrict__ q, const TKV* __restrict__ kpool, const TKV* __restrict__ vpool,
    const int32_t* __restrict__ row_pos, const int32_t* __restrict__ row_slot,
    const int32_t* __restrict__ page_table, TA* __restrict__ o, int nq, int nkv, int d, int pt_stride) {
  __shared__ float s_m[16], s_l[16], s_acc[16][129];
  const int row = blockIdx.x, qh = blockIdx.y, kvh = qh / (nq / nkv);
  const int tid = threadIdx.x, grp = tid >> 4, sub = tid & 15;
  const int pos = row_pos[row], npages = pos / RL_PAGE + 1;
  const int32_t* pt = page_table + (size_t)row_slot[row] * pt_stride;
  auto dim = [&](int j) { return VEC ? (j >> 2) * 64 + sub * 4 + (j & 3) : j * 16 + sub; };
  auto load8 = [&](const auto* p, float (&x)[8]) {     // the lane's dims of one row of d elements
    if constexpr (VEC) {
#pragma unroll
      for (int j = 0; j < 2; j++) {
        const int e = j * 64 + sub * 4;
        x[4 * j] = x[4 * j + 1] = x[4 * j + 2] = x[4 * j + 3] = 0.f;
        if (e < d) ld4(p + e, x[4 * j], x[4 * j + 1], x[4 * j + 2], x[4 * j + 3]);
      }
    } else {
#pragma unroll
      for (int j = 0; j < 8; j++) x[j] = j * 16 + sub < d ? ldf(p + j * 16 + sub) : 0.f;
    }
  };
  float qv[8], acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  load8(q + (size_t)row * nq * d + (size_t)qh * d, qv);
  const float scale = 1.0f / sqrtf((float)d);
  float m = -INFINITY, l = 0.f;
  for (int p0 = 0; p0 < npages; p0 += 4) {
    float k[4][8], v[4][8], sc[4];
#pragma unroll
    for (int u = 0; u < 4; u++) {      // past the end: the last page again, masked below
      const size_t off = (((size_t)pt[min(p0 + u, npages - 1)] * nkv + kvh) * RL_PAGE + grp) * d;
      load8(kpool + off, k[u]);
      load8(vpool + off, v[u]);
    }
    float mx = -INFINITY;
#pragma unroll
    for (int u = 0; u < 4; u++) {
      float dot = 0.f;
#pragma unroll
      for (int j = 0; j < 8; j++) dot += qv[j] * k[u][j];
#pragma unroll
      for (int x = 8; x > 0; x >>= 1) dot += __shfl_xor(dot, x, 16);
      sc[u] = dot * scale;
      if ((p0 + u) * RL_PAGE + grp <= pos) mx = fmaxf(mx, sc[u]);
    }
    const float mn = fmaxf(m, mx);
    const float alpha = m == -INFINITY ? 0.f : expf(m - mn);
    l *= alpha;
#pragma unroll
    for (int j = 0; j < 8; j++) acc[j] *= alpha;
#pragma unroll
    for (int u = 0; u < 4; u++) {
      if ((p0 + u) * RL_PAGE + grp > pos) continue;     // slots behind the row's position may hold anything
      const float pr = expf(sc[u] - mn);
      l += pr;
#pragma unroll
      for (int j = 0; j < 8; j++) acc[j] += pr * v[u][j];
    }
    m = mn;
  }
#pragma unroll
  for (int j = 0; j < 8; j++)
    if (dim(j) < d) s_acc[grp][dim(j)] = acc[j];
  if (sub == 0) { s_m[grp] = m; s_l[grp] = l; }
  __syncthreads();
  if (tid < d) {
    float M = s_m[0];
    for (int g = 1; g < 16; g++) M = fmaxf(M, s_m[g]);
    float L = 0.f, y = 0.f;
    for (int g = 0; g < 16; g++) {
      const float f = s_m[g] == -INFINITY ? 0.f : expf(s_m[g] - M);
      L += f * s_l[g];
      y += f * s_acc[g][tid];
    }
    stf(o + (size_t)row * nq * d + (size_t)qh * d + tid, y / L);
  }
}

template <typename TA>
__global__ void swiglu_kernel(const float* __restrict__ gu, TA* __restrict__ m, int I) {
  int row = blockIdx.y;
  int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= I) return;
  float g = gu[(size_t)row * 2 * I + j], u = gu[(size_t)row * 2 * I + I + j];
  float y = g / (1.0f + expf(-g)) * u;
  stf(m + (size_t)row * I + j, y);
}

// grid (pairs, 2 n_layers): one page of one pool
__global__ void copy_pages_kernel(char* const* __restrict__ pools, const int32_t* __restrict__ pairs, size_t page_bytes) {
  int p = blockIdx.x;
  size_t src = (size_t)pairs[2 * p] * page_bytes, dst = (size_t)pairs[2 * p + 1] * page_bytes;
  char* base = pools[blockIdx.y];
  const uint4* s4 = (const uint4*)(base + src);
  uint4* d4 = (uint4*)(base + dst);
  for (size_t i = threadIdx.x; i < page_bytes / 16; i += blockDim.x) d4[i] = s4[i];
}

__global__ void page_table_update_kernel(int32_t* __restrict__ pt, const int32_t* __restrict__ upd,
                                         int n, int stride) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) pt[(size_t)upd[3 * i] * stride + upd[3 * i + 1]] = upd[3 * i + 2];
}

// ---- launchers ---------------------------------------------------------------------------
template <typename TW>
void launch_embed(hipStream_t s, const TW* E, const int32_t* tok, float* h, int M, int H) {
  if (M > 0) embed_kernel<TW><<<M, 256, 0, s>>>(E, tok, h, H);
}
template void launch_embed<float>(hipStream_t, const float*, const int32_t*, float*, int, int);
template void launch_embed<bf16_t>(hipStream_t, const bf16_t*, const int32_t*, float*, int, int);

template <typename TW, typename TA>
void launch_rmsnorm(hipStream_t s, const float* h, const TW* g, TA* out, int M, int H, float eps) {
  if (M > 0) rmsnorm_kernel<TW, TA><<<M, 256, 0, s>>>(h, g, out, H, eps);
}
template void launch_rmsnorm<float, float>(hipStream_t, const float*, const float*, float*, int, int, float);
template void launch_rmsnorm<bf16_t, bf16_t>(hipStream_t, const float*, const bf16_t*, bf16_t*, int, int, float);

template <typename TA, typename TW>
void launch_gemm_generic(hipStream_t s, const TA* A, const TW* W, float* C, int M, int N, int K,
                         bool accumulate) {
  if (M <= 0) return;
  const bool vec = K % 4 == 0 && ((uintptr_t)A % (4 * sizeof(TA))) == 0 && ((uintptr_t)W % (4 * sizeof(TW))) == 0;
  if (vec) {
    if (M <= 16)
      gemm_mfma32_kernel<TA, TW, 1><<<dim3((N + 15) / 16, 1), 64 * kWaves32, 0, s>>>(A, W, C, M, N, K, accumulate ? 1 : 0);
    else
      gemm_mfma32_kernel<TA, TW, 4><<<dim3((N + 15) / 16, (M + 63) / 64), 64 * kWaves32, 0, s>>>(A, W, C, M, N, K,
                                                                                       accumulate ? 1 : 0);
    return;
  }
  dim3 grid((N + 63) / 64, (M + 63) / 64);
  gemm_generic_kernel<TA, TW><<<grid, 256, 0, s>>>(A, W, C, M, N, K, accumulate ? 1 : 0);
}
template void launch_gemm_generic<float, float>(hipStream_t, const float*, const float*, float*, int, int, int, bool);
template void launch_gemm_generic<bf16_t, bf16_t>(hipStream_t, const bf16_t*, const bf16_t*, float*, int, int, int, bool);

bool norm_gemm32_takes(const void* h, const void* g, const void* W, int K) {
  return K % 4 == 0 && (((uintptr_t)h | (uintptr_t)g | (uintptr_t)W) & 15) == 0;
}
void launch_norm_gemm32(hipStream_t s, float* h, const float* E, const int32_t* tok, const float* g, const float* W, float* C,
                        int M, int N, int K, float eps, bool swiglu) {
  if (M <= 0) return;
  auto go = [&](auto kernel, int rows) {
    kernel<<<dim3((N + 15) / 16, (M + rows - 1) / rows), 64 * kWaves32, 0, s>>>(h, E, tok, g, W, C, M, N, K, eps);
  };
  if (M <= 16) {
    if (swiglu) go(norm_gemm32_kernel<1, true, false>, 16);
    else if (tok) go(norm_gemm32_kernel<1, false, true>, 16);
    else go(norm_gemm32_kernel<1, false, false>, 16);
  } else {
    if (swiglu) go(norm_gemm32_kernel<4, true, false>, 64);
    else if (tok) go(norm_gemm32_kernel<4, false, true>, 64);
    else go(norm_gemm32_kernel<4, false, false>, 64);
  }
}
// A head's weights are at most 128 KB (a workgroup reads them at about 50 GB/s) and no more than four blocks of 16 rows
// read them again.
bool norm_qkv32_takes(const ModelDims& md, int M) { return (md.d == 64 || md.d == 128) && md.d * md.H <= 32768 && M <= 64; }
void launch_norm_qkv32(hipStream_t s, float* h, const float* E, const int32_t* tok, const float* g, const float* W,
                       const float* gq, const float* gk, const float* rope_cs, const int32_t* row_pos, const int32_t* row_slot,
                       const int32_t* page_table, float* qout, KvPool pool, const ModelDims& md, int M) {
  if (M <= 0) return;
  auto go = [&](auto kernel) {
    kernel<<<dim3(md.nq + 2 * md.nkv, (M + 15) / 16), 64 * kWaves32, 0, s>>>(h, E, tok, g, W, gq, gk, rope_cs, row_pos, row_slot, page_table,
                                                                 qout, (float*)pool.k, (float*)pool.v, md.nq, md.nkv, M, md.H,
                                                                 md.eps, md.qk_norm, md.max_pages_per_traj);
  };
  if (md.d == 64) tok ? go(norm_qkv32_kernel<64, true>) : go(norm_qkv32_kernel<64, false>);
  else tok ? go(norm_qkv32_kernel<128, true>) : go(norm_qkv32_kernel<128, false>);
}

// head_dim 128, bf16, MFMA cache layout: grid (M, ceil(heads / 16)), block 256; qkrope_head128 for sixteen lanes a head.
// The bound holds the dividing forms at five waves a SIMD (93 registers; 101 without it).
template <bool FP8, bool UNDIV>
__global__ __launch_bounds__(256, 5) void qkrope128_kernel(const RopeArgs a, const int32_t* __restrict__ row_pos,
                                                           const int32_t* __restrict__ row_slot,
                                                           const int32_t* __restrict__ page_table, bf16_t* __restrict__ qout,
                                                           bf16_t* __restrict__ kpool, bf16_t* __restrict__ vpool, int pt_stride) {
  const int row = blockIdx.x, sub = threadIdx.x & 15;
  const int hd = blockIdx.y * 16 + (threadIdx.x >> 4);
  if (hd >= a.nq + 2 * a.nkv) return;          // whole 16-lane groups leave together; no barrier below
  const int pos = row_pos[row];
  uint2 w1, w2;
  qkrope_head128<FP8, UNDIV>(a, row, hd, sub, pos, [&] { return page_table[(size_t)row_slot[row] * pt_stride + (pos >> 4)]; }, kpool,
                             vpool, &w1, &w2);
  if (hd < a.nq) {
    bf16_t* dst = qout + ((size_t)row * a.nq + hd) * 128 + sub * 4;
    *(uint2*)dst = w1;
    *(uint2*)(dst + 64) = w2;
  }
}

void launch_qkrope128(hipStream_t s, const RopeArgs& a, const int32_t* row_pos, const int32_t* row_slot, const int32_t* page_table,
                      bf16_t* qout, KvPool pool, const ModelDims& md, int M) {
  if (M <= 0) return;
  const dim3 grid(M, (md.nq + 2 * md.nkv + 15) / 16);
  auto go = [&](auto kernel) {
    kernel<<<grid, 256, 0, s>>>(a, row_pos, row_slot, page_table, qout, (bf16_t*)pool.k, (bf16_t*)pool.v, md.max_pages_per_traj);
  };
  if (md.kv_fp8) a.ssq ? go(qkrope128_kernel<true, true>) : go(qkrope128_kernel<true, false>);
  else a.ssq ? go(qkrope128_kernel<false, true>) : go(qkrope128_kernel<false, false>);
}

template <typename TW, typename TA, typename TKV>
void launch_qkrope(hipStream_t s, const float* qkv, const TW* gq, const TW* gk, const float* rope_cs,
                   const int32_t* row_pos, const int32_t* row_slot, const int32_t* page_table, TA* qout,
                   KvPool pool, const ModelDims& md, int M) {
  if (M <= 0) return;
  dim3 grid(M, md.nq + 2 * md.nkv);
  qkrope_kernel<TW, TA, TKV><<<grid, 64, 0, s>>>(qkv, gq, gk, rope_cs, row_pos, row_slot, page_table, qout,
                                                 (TKV*)pool.k, (TKV*)pool.v, md.nq, md.nkv, md.d, md.eps,
                                                 md.qk_norm, md.max_pages_per_traj);
}
template void launch_qkrope<float, float, float>(hipStream_t, const float*, const float*, const float*, const float*, const int32_t*, const int32_t*, const int32_t*, float*, KvPool, const ModelDims&, int);
template void launch_qkrope<bf16_t, bf16_t, bf16_t>(hipStream_t, const float*, const bf16_t*, const bf16_t*, const float*, const int32_t*, const int32_t*, const int32_t*, bf16_t*, KvPool, const ModelDims&, int);

template <typename TA, typename TKV>
void launch_attention_generic(hipStream_t s, const TA* q, KvPool pool, const int32_t* row_pos,
                              const int32_t* row_slot, const int32_t* page_table, TA* o,
                              const ModelDims& md, int M) {
  if (M <= 0) return;
  dim3 grid(M, md.nq);
  if (md.d % 4 == 0)     // rows of whole 4-element pieces: pools and q are allocated on 256-byte boundaries
    attention_generic_kernel<TA, TKV, true><<<grid, 256, 0, s>>>(
        q, (const TKV*)pool.k, (const TKV*)pool.v, row_pos, row_slot, page_table, o, md.nq, md.nkv,
        md.d, md.max_pages_per_traj);
  else
    attention_generic_kernel<TA, TKV, false><<<grid, 256, 0, s>>>(
        q, (const TKV*)pool.k, (const TKV*)pool.v, row_pos, row_slot, page_table, o, md.nq, md.nkv,
        md.d, md.max_pages_per_traj);
}
template void launch_attention_generic<float, float>(hipStream_t, const float*, KvPool, const int32_t*, const int32_t*, const int32_t*, float*, const ModelDims&, int);
template void launch_attention_generic<bf16_t, bf16_t>(hipStream_t, const bf16_t*, KvPool, const int32_t*, const int32_t*, const int32_t*, bf16_t*, const ModelDims&, int);

template <typename TA>
void launch_swiglu(hipStream_t s, const float* gu, TA* m, int M, int I) {
  if (M > 0) swiglu_kernel<TA><<<dim3((I + 255) / 256, M), 256, 0, s>>>(gu, m, I);
}
template void launch_swiglu<float>(hipStream_t, const float*, float*, int, int);
template void launch_swiglu<bf16_t>(hipStream_t, const float*, bf16_t*, int, int);

void launch_copy_pages(hipStream_t s, char* const* pools, int n_layers, const int32_t* pairs, int n_pairs,
                       size_t page_bytes) {
  if (n_pairs <= 0) return;
  copy_pages_kernel<<<dim3(n_pairs, 2 * n_layers), 256, 0, s>>>(pools, pairs, page_bytes);
}
void launch_page_table_update(hipStream_t s, int32_t* page_table, const int32_t* upd, int n,
                              int stride) {
  if (n <= 0) return;
  page_table_update_kernel<<<(n + 255) / 256, 256, 0, s>>>(page_table, upd, n, stride);
}
