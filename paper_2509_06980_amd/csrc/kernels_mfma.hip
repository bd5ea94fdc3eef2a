// bf16 MFMA kernels for gfx950: weight-streaming GEMM, weight repack, paged GQA attention.
// They implement the same decoder pieces as the generic kernels (policy forward of the paper's
// Generate / Update steps, Section 2.3.2) for head_dim 128 and tile-aligned widths.
#include "kernels.h"
#include "qkrope.h"

#include <algorithm>
#include <atomic>
#include <type_traits>

// =============================================================================================
// Weight repack: W[N,K] row-major -> [K/64 chunks][N/32 strips][4 k-blocks][64 lanes][8].  One
// (chunk, strip) cell is 4 KB: four 32x32x16 MFMA column operands in lane order
// (lane = n % 32 + 32 * ((k % 16) / 8), 8 consecutive k per lane).  Chunk-major order makes all
// workgroups that advance through K in step sweep HBM contiguously; a strip-major order puts
// every wave's stream at a multiple of K * 64 bytes and piles them onto a few memory channels.
// =============================================================================================
__global__ void repack_weight_kernel(const bf16_t* __restrict__ W, const bf16_t* __restrict__ Wu,
                                     bf16_t* __restrict__ Wp, int N, int K, int interleave8) {
  size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int NB = N / 32;
  size_t total = (size_t)NB * (K / 16) * 64;
  if (t >= total) return;
  int lane = (int)(t & 63);
  size_t blk = t >> 6;                 // ((chunk * NB + strip) * 4 + k-block in chunk)
  int kb4 = (int)(blk & 3);
  size_t cell = blk >> 2;
  int nb = (int)(cell % NB);
  int chunk = (int)(cell / NB);
  int n = nb * 32 + (lane & 31);
  int k = chunk * 64 + kb4 * 16 + (lane >> 5) * 8;
  const bf16_t* src;
  if (interleave8) {
    int grp = n >> 3;                       // even groups: gate rows, odd groups: up rows
    int srow = (grp >> 1) * 8 + (n & 7);
    src = ((grp & 1) ? Wu : W) + (size_t)srow * K + k;
  } else {
    src = W + (size_t)n * K + k;
  }
  *(uint4*)(Wp + t * 8) = *(const uint4*)src;
}

void launch_repack_weight(hipStream_t s, const bf16_t* W, const bf16_t* Wu, bf16_t* Wp, int N,
                          int K, bool interleave8) {
  size_t total = (size_t)(N / 32) * (K / 16) * 64;
  repack_weight_kernel<<<(unsigned)((total + 255) / 256), 256, 0, s>>>(W, Wu, Wp, N, K,
                                                                        interleave8 ? 1 : 0);
}

// =============================================================================================
// GEMM  C[M,N] = A[M,K] * W[N,K]^T for weight streaming.  Workgroup = 4 waves, tile
// 128 rows x 128 columns; wave w owns the 32-column strip 4*blockIdx.x + w for all 128 rows
// (4 accumulators of 32x32).  Per 64-k chunk the A tile (16 KB, already in operand order in HBM)
// is copied to LDS and shared by the waves; each wave streams its own weight cells straight from
// HBM into registers, two chunks ahead.  blockIdx.z selects a K-slice (split-K); every slice
// stores its own fp32 partial sum, which the consumer kernel adds in a fixed order (no atomics:
// results are bit-reproducible).
// MB = number of 32-row blocks of the tile that can hold rows (1, 2 or 4; the launcher picks the
// smallest that covers M when there is one row tile): only those blocks of the A chunk are
// fetched, staged and multiplied.  At decode sizes a workgroup's time follows the bytes its CU
// fetches, and the A chunk is half of them, so small batches gain most of what they leave out
// (N = 4096 K = 12288 in eight slices: 22.9 us with all four row blocks, 18.4 at 12 rows, 20.3 at 64; lm-head
// 151936 x 2560 151 -> 137 us at 12 rows, 154 -> 145 at 48, plain loads; past the caches 127 at 12); results per row are
// unchanged.
// EPI_SWIGLU and EPI_LSE form the product transposed; see swiglu_block.  UNDIV (EPI_SWIGLU): the rows of A are still to be
// divided by their rms, zt holds their sums of squares and scale_c is epsilon (see gemm_residual_kernel).  A choice at compile
// time: tested at run time the division had grown the plain form from 7.4 to 13.3 KB of code with four row blocks.
// EPI_LSE (lm-head of the masked log-prob pass): the product is formed transposed (weights as the
// MFMA row operand; both operands have the same lane layout, so swapping them costs nothing), which
// puts 16 vocabulary entries of one batch row into the registers of a lane.  The epilogue reduces
// its 32-column strip per row to (max, sum of 2^((z - max) c)) and picks out the target token's
// logit; the logits themselves are never stored.
// EPI_STORE_MAX (lm-head of a decode step): EPI_STORE plus, per row, the maximum over the wave's 32
// columns (a butterfly over the 32 lanes of each half that halves the values a lane holds at every
// step), written to zt[row * (N / 32) + strip]: the sampler gets the row maximum it needs before
// any weight can be formed from V / 32 numbers per row instead of a pass over the logits.
// =============================================================================================
// Sum of p[x * stride] over x = first, first + step, ... below n, in ascending order, eight reads in flight (a loop with
// one read at a time is a chain of latencies: 64 of them 2.4 us).
__device__ __forceinline__ float strided_sum(const float* __restrict__ p, int first, int step, int n, int stride) {
  float t = 0.f;
  for (int x = first; x < n; x += 8 * step) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; u++) v[u] = p[min(x + u * step, n - 1) * stride];
#pragma unroll
    for (int u = 0; u < 8; u++) t += x + u * step < n ? v[u] : 0.f;
  }
  return t;
}

// SwiGLU of one transposed 32x32 block (EPI_SWIGLU forms the product with the weights as the row
// operand): lane l holds, for batch row l % 32, weight rows (i / 4) * 8 + (l / 32) * 4 + i % 4, and the
// repack puts 8 gate rows before the 8 up rows of the same units: gate and up of a unit are in the same
// lane (registers i and i + 4), every lane works, and four consecutive units leave as one 8-byte store
// (32 rows x 16 bytes of the A-tile layout contiguous).  With gate and up in different lanes, half the
// lanes idle and 2-byte stores the epilogue had cost 24 us per round of 256 x 256 tiles.
template <typename F>
__device__ __forceinline__ void swiglu_block(F val, bf16_t* __restrict__ out, int row, int M, int nb, int lane,
                                             int width) {
  if (row >= M) return;
#pragma unroll
  for (int p = 0; p < 2; p++) {
    uint32_t y[4];
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const float v = val(8 * p + e), u = val(8 * p + 4 + e);
      y[e] = f2bf(v / (1.0f + __expf(-v)) * u);
    }
    *(uint2*)(out + atile_off(row, nb * 16 + p * 8 + (lane >> 5) * 4, width)) =
        make_uint2(y[0] | (y[1] << 16), y[2] | (y[3] << 16));
  }
}
// Log-softmax statistics of one transposed 32x32 block: lane l holds 16 vocabulary entries of batch row
// l % 32; its half of the strip and the other lane half's are joined with one swap.
template <typename F>
__device__ __forceinline__ void lse_block(F val, float2* __restrict__ P, float* __restrict__ zt,
                                          const int32_t* __restrict__ tgt, int row, int M, int nb, int NB, int lane,
                                          float scale_c) {
  float mx = val(0);
#pragma unroll
  for (int i = 1; i < 16; i++) mx = fmaxf(mx, val(i));
  mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
  float sm = 0.f;
#pragma unroll
  for (int i = 0; i < 16; i++) sm += exp2f((val(i) - mx) * scale_c);
  sm += __shfl_xor(sm, 32, 64);
  if (row >= M) return;
  if (lane < 32) P[(size_t)row * NB + nb] = make_float2(mx, sm);
  const int t = tgt[row];
  if ((t >> 5) == nb && ((t >> 2) & 1) == (lane >> 5)) {
    const int isel = ((t & 31) >> 3) * 4 + (t & 3);
    float z = val(0);
#pragma unroll
    for (int i = 1; i < 16; i++) z = isel == i ? val(i) : z;
    zt[row] = z;
  }
}

// Weights that are read once a pass and are too large to stay in the 256 MB last-level cache until the next one go past
// the caches.  The line: products of 31 MB and more gain 3 to 7 % from it at 64 rows and fewer (see the kernels), one of
// 21 MB nothing, and those of a model that the cache holds (4 MB, 64 of them in turn) lose up to 30 % (3.0 -> 3.9 us).
static bool streams_weights(int N, int K) { return (size_t)N * K * 2 >= ((size_t)24 << 20); }

template <int EPI, int MB, bool NT, bool UNDIV = false>
__global__ __launch_bounds__(256) void gemm_mfma_kernel(const bf16_t* __restrict__ A,
                                                        const bf16_t* __restrict__ Wp,
                                                        void* __restrict__ Cv, int M, int N,
                                                        int K, int chunks_per_split,
                                                        const int32_t* __restrict__ tgt,
                                                        float* __restrict__ zt, float scale_c) {
  // a thread stages MB 16-byte pieces of the used part of an A chunk
  __shared__ u32x4 As[2][1024];
  __shared__ float sq[UNDIV ? 256 : 1];      // [half of the partial sums][row]
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int nb = blockIdx.x * 4 + wave;
  const bool active = nb * 32 < N;
  const int mt = blockIdx.y;
  const int nchunks = K >> 6;
  const int c0 = blockIdx.z * chunks_per_split;
  const int c1 = min(c0 + chunks_per_split, nchunks);
  const u32x4* Ag = (const u32x4*)(A + (size_t)mt * K * 128);       // tile: 128 rows x K
  // piece p of the used part of a chunk -> its offset in the chunk (k-block, row block, lane):
  // with MB < 4 only the first MB row blocks of every k-block are staged
  auto a_piece = [](int p) { return MB == 4 ? p : (p / (64 * MB)) * 256 + (p % (64 * MB)); };
  const int NB = N >> 5;
  const u32x4* Wg = (const u32x4*)Wp + (size_t)(active ? nb : 0) * 256;   // cell (chunk 0, strip nb)
  // NT (at most 64 rows: one row tile, every weight read once, the stream from HBM is all that counts): past the caches.
  // lm-head of 151936 x 4096 at 6 rows 212 -> 190 us (6.5 TB/s), x 2560 at 37 rows 144 -> 135, x 1024 at one row 54 ->
  // 51.5; N = 4096 K = 12288 in eight slices at 6 rows 19.1 -> 17.8.  At 128 rows the kernel is not held by the stream
  // and plain loads are the better ones (164 against 166 us).
  auto weight = [](const u32x4* p) {
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
  };
  f32x16 acc[MB];
#pragma unroll
  for (int i = 0; i < MB; i++)
#pragma unroll
    for (int j = 0; j < 16; j++) acc[i][j] = 0.f;
  // Two chunks of A (for the whole workgroup) and of this wave's weight strip are kept in flight
  // (fewer registers and more resident workgroups than with four: measured best at M = 128).
  // Loads past the end of the K-slice are clamped to its last chunk (re-reads that hit in L2) so
  // that the pipeline has no conditional register definitions.  Stages are spelled out (no
  // arrays of stages) so that every buffer lives in registers.
  const int clast = c1 - 1;
  u32x4 a0[MB], a1[MB], b0[4], b1[4];
#define GEMM_LOAD(AR, BR, CHUNK)                                            \
  {                                                                         \
    const int cl_ = min((CHUNK), clast);                                    \
    _Pragma("unroll") for (int i = 0; i < MB; i++)                          \
      AR[i] = Ag[(size_t)cl_ * 1024 + a_piece(i * 256 + tid)];              \
    _Pragma("unroll") for (int i = 0; i < 4; i++)                           \
      BR[i] = weight(Wg + ((size_t)cl_ * NB * 4 + i) * 64 + lane);          \
    /* keep the scheduler from sinking these loads towards their use */     \
    __builtin_amdgcn_sched_barrier(0);                                      \
  }
#define GEMM_STAGE(S, AR, BR)                                               \
  {                                                                         \
    const int cc = c + (S);                                                 \
    u32x4* buf = As[S];                                                     \
    /* past the end of the slice the weight operand is zeroed: the body stays branch free; \
       the masked copy also frees the staging registers before they are refilled */ \
    const unsigned keep = cc < c1 ? 0xffffffffu : 0u;                       \
    u32x4 bcur[4];                                                          \
    _Pragma("unroll") for (int i = 0; i < MB; i++) buf[a_piece(i * 256 + tid)] = AR[i]; \
    _Pragma("unroll") for (int i = 0; i < 4; i++) bcur[i] = BR[i] & keep;   \
    __builtin_amdgcn_sched_barrier(0);                                      \
    __syncthreads();                                                        \
    GEMM_LOAD(AR, BR, cc + 2)                                               \
    /* all 16 row operands of the chunk are requested from LDS before the first MFMA: with one \
       wave per SIMD nothing else hides the LDS latency */                  \
    u32x4 av[16];                                                           \
    _Pragma("unroll") for (int i = 0; i < 16; i++) if ((i & 3) < MB) av[i] = buf[i * 64 + lane]; \
    __builtin_amdgcn_sched_barrier(0);                                      \
    _Pragma("unroll") for (int kk = 0; kk < 4; kk++) {                      \
      bf16x8 b = __builtin_bit_cast(bf16x8, bcur[kk]);                      \
      _Pragma("unroll") for (int mb = 0; mb < MB; mb++) {                   \
        bf16x8 a = __builtin_bit_cast(bf16x8, av[kk * 4 + mb]);             \
        acc[mb] = EPI == EPI_LSE || EPI == EPI_SWIGLU                       \
                      ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, a, acc[mb], 0, 0, 0) \
                      : __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[mb], 0, 0, 0); \
      }                                                                     \
    }                                                                       \
  }
  GEMM_LOAD(a0, b0, c0)
  GEMM_LOAD(a1, b1, c0 + 1)
  if (UNDIV) {
    // A thread sums two of a row's four interleaved shares of partial sums, in the order of gemm_decode_kernel, while the
    // first chunks arrive; the epilogue reads both halves from LDS, behind the loop's barriers.  Summed in the epilogue,
    // by every wave for itself and one row block after the other, they cost 4 to 6 us (gate-up of hidden 1024 at 131 rows,
    // undivided rows or not: 20.3 and 13.8 us, now 15.5; of hidden 512 at 300 rows 13.0 and 8.8, now 9.8).
    const int q = (tid >> 7) * 2, n = K >> 4, r16 = (M + 15) >> 4 << 4;
    const float* p = zt + min(mt * 128 + (tid & 127), M - 1);
    float t0 = 0.f, t1 = 0.f;
    for (int x = q; x < n; x += 32) {      // n is a multiple of 4
      float v[16];
#pragma unroll
      for (int u = 0; u < 8; u++) {
        const float* px = p + (size_t)min(x + 4 * u, n - 4 + q) * r16;
        v[2 * u] = px[0];
        v[2 * u + 1] = px[r16];
      }
#pragma unroll
      for (int u = 0; u < 8; u++) {
        t0 += x + 4 * u < n ? v[2 * u] : 0.f;
        t1 += x + 4 * u < n ? v[2 * u + 1] : 0.f;
      }
    }
    sq[tid] = t0 + t1;
  }
  // the barrier inside a stage also orders its LDS store after every wave's reads of the same
  // buffer two chunks earlier
  for (int c = c0; c < c1; c += 2) {
    GEMM_STAGE(0, a0, b0)
    GEMM_STAGE(1, a1, b1)
  }
#undef GEMM_LOAD
#undef GEMM_STAGE
  if (!active) return;
  if (EPI == EPI_LSE || EPI == EPI_SWIGLU) {
    // acc[mb][i] belongs to batch row mb*32 + lane%32 and weight row nb*32 + (i/4)*8 + (lane/32)*4 + i%4
#pragma unroll
    for (int mb = 0; mb < MB; mb++) {
      const int row = mt * 128 + mb * 32 + (lane & 31);
      float inv = 1.0f;
      if (UNDIV) {
        const float* t = sq + mb * 32 + (lane & 31);
        inv = 1.0f / sqrtf((t[0] + t[128]) / (float)K + scale_c);
      }
      auto val = [&](int i) { return UNDIV ? acc[mb][i] * inv : acc[mb][i]; };
      if (EPI == EPI_SWIGLU) swiglu_block(val, (bf16_t*)Cv, row, M, nb, lane, N >> 1);
      else lse_block(val, (float2*)Cv, zt, tgt, row, M, nb, NB, lane, scale_c);
    }
    return;
  }
  const int col = nb * 32 + (lane & 31);
  float* Cp = (float*)Cv + (size_t)blockIdx.z * M * N;
  if (EPI == EPI_STORE_MAX) {
    // v[j], j = 16 mb + i, is the value of row mt*128 + 32 mb + (i>>2)*8 + (lane>>5)*4 + (i&3) in
    // this lane's column.  Step s pairs lanes L and L ^ (1 << s): of every two values the lane
    // with bit s clear keeps the even one, the other lane the odd one, and each takes the maximum
    // with what its partner held of the kept one.  After the five steps lane L holds the strip
    // maxima of the values j = 32 k + (L & 31).
    float v[16 * MB];
#pragma unroll
    for (int mb = 0; mb < MB; mb++)
#pragma unroll
      for (int i = 0; i < 16; i++) v[mb * 16 + i] = acc[mb][i];
    int n = 16 * MB;
#pragma unroll
    for (int st = 0; st < 5; st++) {
      const bool up = (lane >> st) & 1;
      if (n >= 2) {
        n >>= 1;
#pragma unroll
        for (int k = 0; k < 32; k++)
          if (k < n) {
            const float keep = up ? v[2 * k + 1] : v[2 * k];
            const float send = up ? v[2 * k] : v[2 * k + 1];
            v[k] = fmaxf(keep, __shfl_xor(send, 1 << st, 64));
          }
      } else {
        v[0] = fmaxf(v[0], __shfl_xor(v[0], 1 << st, 64));
      }
    }
    constexpr int NOUT = MB == 4 ? 2 : 1;
    const int jl = MB == 1 ? (lane & 15) : (lane & 31);
    if (MB > 1 || (lane & 16) == 0) {
#pragma unroll
      for (int k = 0; k < NOUT; k++) {
        const int j = 32 * k + jl, mb = j >> 4, i = j & 15;
        const int row = mt * 128 + mb * 32 + (i >> 2) * 8 + (lane >> 5) * 4 + (i & 3);
        if (row < M) zt[(size_t)row * NB + nb] = v[k];
      }
    }
  }
#pragma unroll
  for (int mb = 0; mb < MB; mb++) {
#pragma unroll
    for (int i = 0; i < 16; i++) {
      int row = mt * 128 + mb * 32 + (i >> 2) * 8 + (lane >> 5) * 4 + (i & 3);
      float v = acc[mb][i];
      if (row < M) {
        __builtin_nontemporal_store(v, &Cp[(size_t)row * N + col]);   // leaves the L2 early instead of at the end of the kernel
      }
    }
  }
}

// =============================================================================================
// GEMM for many rows (chunked prefill, teacher-forced passes, mixed steps): tile 64*MB x 64*NBW, 4 waves
// as 2 x 2, wave tile 32*MB x 32*NBW (MB = 4: 256 rows; NBW = 4: 256 columns, 16 accumulators of 32x32;
// NBW = 5: 320 columns, 20 of them; MB = 2, NBW = 4: 128 x 256, for passes of a few hundred rows, whose last
// 256-row tile would be mostly empty).  Per 16-k step a wave reads MB row and NBW column operands from
// LDS for MB*NBW MFMAs.
// Both operands go from memory straight into LDS (16-byte buffer loads with the LDS destination; no
// staging registers, no LDS stores in the instruction stream) as chunks of 32 k in a ring of R stages.  The
// loads return in order, so "at most the chunks behind it outstanding" means that the next chunk has landed;
// before the epilogue all are drained.  Chunks behind the slice and 32-row blocks without rows are asked for behind the
// buffer's end: zeros, no memory traffic.
// MB = 4: four stages, three and a half chunks ahead, operands one 16-k step ahead.  Every group of NBW MFMAs carries its share of
// the loads, and the next step's operands are read ahead of its last group, so that the wait in front of the barrier
// (half way through a chunk: the next chunk is complete, this one is read out) finds them there.
// What bounds it at thousands of rows is power: on operands of zeros the same instructions take 213 us instead of 295
// (8192 x 2560 x 9728: 1.92 and 1.38 PFLOP/s), and MFMAs alone, on registers, reach 2.4 and 1.87.  (16x16x32 MFMAs
// draw less, 2.13 PFLOP/s alone with two waves a SIMD, but one wave a SIMD cannot issue them back to back: 312 us.)
// MB = 2: bound by what the CUs fetch from L2 (without the loads 587 x 2560 x 9728 in five slices takes 27 us of 35; matrix pipes 0.36 of
// the time busy, addressers 0.60) and by the latencies of one wave a SIMD: the operands of a whole chunk are read one chunk ahead, one
// read behind an MFMA, and the next chunk's loads between them (587 x 2560 x 4096 undivided, 50 workgroups: 51 us with operands half a chunk ahead, reads and
// loads in front of each group of four MFMAs; 43.5 a chunk ahead; 41.4 one by one).  Three stages let two workgroups share a CU;
// where there is only one to a CU anyway four hide more of the weights' stream (300 x 19456 x 2560 42.6 -> 39.7 us).
// The fifth accumulator column lives in vector registers: 320 accumulator registers exceed the 256
// accumulation registers, and the builtin, which takes all of its kind from one file, then copies.
// A K-slice (EPI_STORE only) stores its own partial sum.
// The k order per output element is that of the 128 x 128 kernel: with one slice the bits are the same.
// EPI_QKV / EPI_QKV8 (bf16 / 8-bit cache; NBW = 4: a wave's 128 columns are one head): the product is
// formed transposed, which leaves a row's 128 dims of the head in two lanes, RoPE partners in the
// same lane; the per-head norm (one swap), RoPE and the writes to q and the paged cache happen in
// the epilogue, so the fp32 projection (201 MB at 8192 x 6144) is neither stored nor read back.
// EPI_ADD: the product is added to the fp32 residual stream in place (O and down, one slice): 13 to 19 us more
// than storing it at 8192 x 2560 (84 MB read by all workgroups at once), 30 us less in the norm behind it.
// Measured at 8192 rows (us alone / in the pass; before: register staging, 256-column tiles or 128 x 128, in the
// pass): gate-up N = 19456 K = 2560 with SwiGLU 880 -> 646 / 655 (1.26 PFLOP/s), down N = 2560 K = 9728 443 -> 296
// stored (1.38 PFLOP/s), 315 / 316 added, O N = 2560 K = 4096 192 -> 132 stored, 146 / 153 added, QKV N = 6144 K = 2560
// with norm, RoPE and cache write 244 + 80 -> 247 / 264, lm-head with log-softmax at 1536 rows (N = 151936) 1709 ->
// 1015 / 986.
// XCD-aware tile numbering (xcd_tile).  K % 64 == 0, N % 32 == 0.
// =============================================================================================
// Tile and K-slice of a workgroup: the hardware hands workgroups to the 8 XCDs round-robin by linear index
// and each XCD has its own L2.  XCD x works through a contiguous range of a sequence that takes one slice after the
// other and in it groups of gm_most row tiles column by column, so the 32 workgroups resident on an XCD cover a
// compact block of tiles of one slice (256-row tiles: 4 x 8, 12 distinct operand tiles per chunk instead of ~22).  With
// the slices dealt over all XCDs an XCD had met a few tiles of every slice (128 x 256 tiles, 587 x 2560 x 9728 in five
// slices 36.7 -> 35.2 us, 300 rows in eight 25.7 -> 23.8).  A bijection for any tile counts.
__device__ __forceinline__ void xcd_tile(int gm_most, int* tm, int* tn, int* slice) {
  const int tiles_n = gridDim.x, tiles_m = gridDim.y, tiles = tiles_m * tiles_n, total = tiles * gridDim.z;
  const int id = (blockIdx.z * tiles_m + blockIdx.y) * tiles_n + blockIdx.x;
  const int base = total >> 3, rem = total & 7, x = id & 7;
  const int vid = x * base + min(x, rem) + (id >> 3), z = vid / tiles, v = vid - z * tiles;
  const int per_group = gm_most * tiles_n, grp = v / per_group, first = grp * gm_most;
  const int gm = min(gm_most, tiles_m - first), within = v - grp * per_group;
  // the divisions leave them in vector registers
  *tm = __builtin_amdgcn_readfirstlane(first + within % gm);
  *tn = __builtin_amdgcn_readfirstlane(within / gm);
  *slice = __builtin_amdgcn_readfirstlane(z);
}

// QK-norm, RoPE and the writes of one head (EPI_QKV) for a wave's MB blocks of 32 batch rows:
// val(a, b, i) is dim 32 b + (i / 4) * 8 + (lane / 32) * 4 + i % 4 of the head for row row0 + 32 a + lane % 32.
// The same arithmetic as qkrope128_kernel; only the order of the sum of squares differs.  With one wave
// per SIMD nothing else hides a memory round trip: positions, pages and gains are read once, and the
// RoPE table pieces of half a row block are requested before the half ahead of it is computed.
template <bool FP8, int MB, typename F>
__device__ __forceinline__ void qkv_head(F val, const QkvArgs& q, int row0, int M, int hd, int lane) {
  const int h4 = (lane >> 5) * 4;
  const bool is_q = hd < q.nq, is_v = hd >= q.nq + q.nkv;
  int pos[MB];
  size_t blk[MB];
#pragma unroll
  for (int a = 0; a < MB; a++) pos[a] = q.row_pos[min(row0 + 32 * a + (lane & 31), M - 1)];
#pragma unroll
  for (int a = 0; a < MB; a++) {
    blk[a] = 0;
    if (!is_q) {
      const int slot = q.row_slot[min(row0 + 32 * a + (lane & 31), M - 1)];
      const int page = q.page_table[(size_t)slot * q.pt_stride + (pos[a] >> 4)];
      blk[a] = ((size_t)page * q.nkv + (is_v ? hd - q.nq - q.nkv : hd - q.nq)) * (RL_PAGE * 128);
    }
  }
  if (is_v) {
#pragma unroll
    for (int a = 0; a < MB; a++) {
      if (row0 + 32 * a + (lane & 31) >= M) continue;
      const int tok = pos[a] & (RL_PAGE - 1);
#pragma unroll
      for (int b = 0; b < 4; b++)
#pragma unroll
        for (int i = 0; i < 16; i++) {
          const int d = 32 * b + (i >> 2) * 8 + h4 + (i & 3);
          if (FP8) ((uint8_t*)q.vpool)[blk[a] + vswz8_off(tok, d)] = f2e4m3(val(a, b, i));
          else ((bf16_t*)q.vpool)[blk[a] + vswz_off(tok, d)] = f2bf(val(a, b, i));
        }
      __builtin_amdgcn_sched_barrier(0);
    }
    return;
  }
  const bf16_t* g = is_q ? q.gq : q.gk;
  uint2 gl[8], gh[8];      // gains of dims 32 b + 8 c + h4 .. + 3 and of their partners, piece x = 4 b + c
#pragma unroll
  for (int x = 0; x < 8; x++) {
    const int d = 32 * (x >> 2) + (x & 3) * 8 + h4;
    gl[x] = gh[x] = make_uint2(0u, 0u);
    if (q.qk_norm) {
      gl[x] = *(const uint2*)(g + d);
      gh[x] = *(const uint2*)(g + d + 64);
    }
  }
  float4 cs[2][8];         // (cos, sin) of four pieces: half a row block, y = 2 a + b
  auto fetch = [&](int y) {
#pragma unroll
    for (int c = 0; c < 4; c++) {
      const float* t = q.rope_cs + ((size_t)pos[y >> 1] * 64 + 32 * (y & 1) + c * 8 + h4) * 2;
      cs[y & 1][2 * c] = *(const float4*)t;
      cs[y & 1][2 * c + 1] = *(const float4*)(t + 4);
    }
  };
  fetch(0);
  float inv = 1.0f;
#pragma unroll
  for (int y = 0; y < 2 * MB; y++) {
    const int a = y >> 1, b = y & 1;
    if (y < 2 * MB - 1) fetch(y + 1);
    __builtin_amdgcn_sched_barrier(0);
    if (b == 0) {
      float ss = 0.f;
#pragma unroll
      for (int v = 0; v < 4; v++)
#pragma unroll
        for (int i = 0; i < 16; i++) {
          const float x = val(a, v, i);
          ss += x * x;
        }
      ss += __shfl_xor(ss, 32, 64);
      inv = 1.0f / sqrtf(ss / 128.0f + q.eps);
      __builtin_amdgcn_sched_barrier(0);
    }
    const int row = row0 + 32 * a + (lane & 31), tok = pos[a] & (RL_PAGE - 1);
    if (row < M) {
#pragma unroll
      for (int c = 0; c < 4; c++) {
        const int x = 4 * b + c, d = 32 * b + c * 8 + h4;
        const float4 c0 = cs[y & 1][2 * c], c1 = cs[y & 1][2 * c + 1];
        const float co[4] = {c0.x, c0.z, c1.x, c1.z}, sn[4] = {c0.y, c0.w, c1.y, c1.w};
        float y1[4], y2[4];
#pragma unroll
        for (int e = 0; e < 4; e++) {
          float x1 = val(a, b, 4 * c + e), x2 = val(a, b + 2, 4 * c + e);
          if (q.qk_norm) {
            x1 = x1 * inv * bf2f((bf16_t)((e & 2 ? gl[x].y : gl[x].x) >> (e & 1 ? 16 : 0)));
            x2 = x2 * inv * bf2f((bf16_t)((e & 2 ? gh[x].y : gh[x].x) >> (e & 1 ? 16 : 0)));
          }
          y1[e] = x1 * co[e] - x2 * sn[e];
          y2[e] = x2 * co[e] + x1 * sn[e];
        }
        if (FP8 && !is_q) {
          uint8_t* k8 = (uint8_t*)q.kpool + blk[a];
          *(uint32_t*)(k8 + kswz8_off(tok, d)) = f2e4m3x4(y1[0], y1[1], y1[2], y1[3]);
          *(uint32_t*)(k8 + kswz8_off(tok, d + 64)) = f2e4m3x4(y2[0], y2[1], y2[2], y2[3]);
          continue;
        }
        const uint2 w1 = make_uint2((uint32_t)f2bf(y1[0]) | ((uint32_t)f2bf(y1[1]) << 16),
                                    (uint32_t)f2bf(y1[2]) | ((uint32_t)f2bf(y1[3]) << 16));
        const uint2 w2 = make_uint2((uint32_t)f2bf(y2[0]) | ((uint32_t)f2bf(y2[1]) << 16),
                                    (uint32_t)f2bf(y2[2]) | ((uint32_t)f2bf(y2[3]) << 16));
        if (is_q) {
          bf16_t* dst = q.qout + ((size_t)row * q.nq + hd) * 128 + d;
          *(uint2*)dst = w1;
          *(uint2*)(dst + 64) = w2;
        } else {
          bf16_t* kb = (bf16_t*)q.kpool + blk[a];
          *(uint2*)(kb + kswz_off(tok, d)) = w1;
          *(uint2*)(kb + kswz_off(tok, d + 64)) = w2;
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Buffer descriptor of `bytes` bytes at p in scalar registers (p and bytes are the same in every lane).
__device__ __forceinline__ u32x4 buffer_rsrc(const void* p, unsigned bytes) {
  const uint64_t a = (uint64_t)p;
  u32x4 r;
  r[0] = __builtin_amdgcn_readfirstlane((unsigned)a);
  r[1] = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32) & 0xffffu);
  r[2] = __builtin_amdgcn_readfirstlane(bytes);
  r[3] = 0x00027000u;
  return r;
}
// One load of 16 bytes per lane straight into LDS (lane l's piece at lds + 16 l).  Inline assembly: after
// the builtin the compiler waits for all such loads before any LDS read.  Whoever uses it waits with an
// explicit vmcnt (the loads return in order), puts a barrier before other waves read, and drains all of
// them before the workgroup ends.  Pieces whose offset lies behind the buffer's end arrive as zeros.
// The compiler counts no wait states for the instructions in here: the scalar operands come from scalar
// arithmetic (one that a vector instruction wrote would have to be five wait states old).
template <bool NT = false>     // past the caches
__device__ __forceinline__ void load_to_lds(unsigned lds, int voff, u32x4 rsrc, unsigned soff) {
  if constexpr (NT)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds" ::"s"(lds), "v"(voff), "s"(rsrc),
               "s"(soff)
               : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds), "v"(voff), "s"(rsrc),
               "s"(soff)
               : "memory", "m0");
}

// Scalar offsets of a workgroup's 1 KB loads: inside the two buffers whatever is asked for.  The hardware compares a lane's
// offset with the buffer's size less the scalar one, so only a lane's offset may lie behind the end.
struct ManyRowLoads {
  int c1, NB, strip0;        // end of the K-slice in chunks of 32 k, strips of the weights, first strip of the tile
  unsigned tile1;            // of the second 128-row tile of the rows, 0 where there is none
  __host__ __device__ int inside(int chunk) const { return chunk < c1 ? chunk : c1 - 1; }
  __host__ __device__ unsigned rows(int chunk, int tile, int kb, int wave) const {
    return (tile ? tile1 : 0u) + (unsigned)((2 * inside(chunk) + kb) * 4 + wave) * 1024u;
  }
  // strips past the end (N not a multiple of the tile): the last one again, results dropped
  __host__ __device__ unsigned weights(int chunk, int j, int wave) const {
    const int c = inside(chunk), s = strip0 + 2 * j + (wave >> 1), st = s < NB ? s : NB - 1;
    return ((unsigned)(c >> 1) * NB + st) * 4096u + (c & 1) * 2048u + (wave & 1) * 1024u;
  }
};

template <int EPI, int MB, int NBW, int R>
__global__ __launch_bounds__(256, MB == 2 && R == 3 ? 2 : 1) void gemm_dma_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ Wp,
                                                       void* __restrict__ Cv, int M, int N, int K,
                                                       int chunks_per_split, const int32_t* __restrict__ tgt,
                                                       float* __restrict__ zt, float scale_c, QkvArgs qkv) {
  constexpr bool TR = EPI != EPI_STORE && EPI != EPI_ADD;   // weights as the row operand
  constexpr int NS = 2 * NBW;                 // strips of the tile
  constexpr int NA = 4 * MB;                  // row pieces of a stage: [128-row tile][kb][32-row block]
  constexpr int PW = MB + NBW;                // 1 KB pieces per wave and chunk
  constexpr int BUF = (NA + 4 * NBW) * 1024;  // bytes of a stage: the row pieces, then [strip][kb]
  constexpr int F = PW / 2;                   // MB = 4: pieces of a chunk that are asked for half a chunk ahead of the others
  constexpr int kFar = 0x7fff0000;            // a lane's offset behind every buffer's end: zeros, no memory traffic
  extern __shared__ u32x4 smem[];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int wm = wave >> 1, wn = wave & 1;
  const int NB = N >> 5, nch = K >> 5, r32 = (M + 31) >> 5;
  int bx, by, slice;
  xcd_tile(MB == 4 ? 4 : 8, &by, &bx, &slice);
  const int c0 = slice * chunks_per_split, c1 = min(c0 + chunks_per_split, nch);
  const int blk0 = by * 2 * MB, strip0 = bx * NS;           // first 32-row block and strip of the tile
  const int mt0 = blk0 >> 2, mts = min((r32 + 3) / 4 - mt0, MB == 4 ? 2 : 1);      // its 128-row tiles of A
  const u32x4 ra = buffer_rsrc(A + (size_t)mt0 * K * 128, (unsigned)mts * (unsigned)K * 256u);
  const u32x4 rb = buffer_rsrc(Wp, (unsigned)N * (unsigned)K * 2u);
  const ManyRowLoads at{c1, NB, strip0, mts > 1 ? (unsigned)K * 256u : 0u};
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void*)smem;
  const int voff = lane * 16;
  int avoff[2];                               // MB = 4: of this wave's row block in either 128-row tile
#pragma unroll
  for (int t = 0; t < 2; t++) avoff[t] = blk0 + 4 * t + wave < r32 ? voff : kFar;
  // piece j of this wave of a chunk into stage buf; chunks behind the slice: the last one's offset, and far = kFar (MB = 4: the last
  // chunk again, never read, as the registers that the choice takes would spill)
  auto dma = [&](int chunk, int j, int buf, int far) {
    const unsigned dst = lds0 + (unsigned)buf * BUF + (unsigned)(j * 4 + wave) * 1024u;
    if (j < MB)
      load_to_lds(dst, MB == 4 ? avoff[j >> 1] : voff | (blk0 + wave < r32 ? far : kFar), ra, at.rows(chunk, j >> 1, j & 1, wave));
    else
      load_to_lds(dst, voff | far, rb, at.weights(chunk, j - MB, wave));
  };
  auto behind = [&](int c) { return MB == 4 || c < c1 ? 0 : kFar; };
  f32x16 acc[MB][4], acc5[MB];
#pragma unroll
  for (int a = 0; a < MB; a++)
#pragma unroll
    for (int e = 0; e < 16; e++) {
      acc5[a][e] = 0.f;
#pragma unroll
      for (int b = 0; b < 4; b++) acc[a][b][e] = 0.f;
    }
  auto mfma = [&](const u32x4& row, const u32x4& col, f32x16& c) {
    c = TR ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, col), __builtin_bit_cast(bf16x8, row), c, 0, 0, 0)
           : __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, row), __builtin_bit_cast(bf16x8, col), c, 0, 0, 0);
  };
  const u32x4* As = smem + (MB == 4 ? wm * 8 : wm * 2) * 64 + lane;   // [kb][32-row block]
  const u32x4* Bs = smem + (NA + wn * NBW * 2) * 64 + lane;           // [strip][kb]
#pragma unroll
  for (int c = 0; c < R - 1; c++)
#pragma unroll
    for (int j = 0; j < PW; j++) dma(c0 + c, j, c, behind(c0 + c));
  if constexpr (MB == 4) {
    u32x4 av[2][MB], bv[2][NBW];
#pragma unroll
    for (int j = 0; j < F; j++) dma(c0 + R - 1, j, R - 1, behind(c0 + R - 1));
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((R - 2) * PW + F) : "memory");
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int x = 0; x < MB; x++) av[0][x] = As[x * 64];
#pragma unroll
    for (int x = 0; x < NBW; x++) bv[0][x] = Bs[x * 128];
    for (int c = c0; c < c1; c++) {
      const int sc = (c - c0) & (R - 1), sn = (sc + 1) & (R - 1), sl = (sc - 1) & (R - 1);      // stages of chunks c, c + 1, c + R - 1
      const int f0 = behind(c + R - 1), f1 = behind(c + R);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int g = 0; g < 2 * MB; g++) {
        const int a = g % MB, st = g / MB;
        if (g == MB) {     // chunk c + 1 has landed for every wave, chunk c is read out by every wave
          asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((R - 2) * PW) : "memory");
          __builtin_amdgcn_s_barrier();
        }
        const int base = (st == 0 ? sc : sn) * (BUF / 16), kb = st == 0 ? 1 : 0;
        auto rd = [&](int q) {      // operand q of the next 16-k step
          if (q < MB) av[1 - st][q] = As[base + (kb * 4 + q) * 64];
          else bv[1 - st][q - MB] = Bs[base + ((q - MB) * 2 + kb) * 64];
        };
        if (a == 0) { rd(4); rd(0); rd(5); }
        if (a == 1) { rd(6); rd(7); rd(1); }
        if (a == 2) { rd(2); rd(3); if (NBW == 5) rd(8); }
        // this step's share of the loads: the rest of chunk c + R - 1, then the first F pieces of chunk c + R
#pragma unroll
        for (int j = 0; j < PW; j++) {
          if (st == 0 && j >= F && (j - F) * MB / (PW - F) == a) dma(c + R - 1, j, sl, f0);
          if (st == 1 && j < F && j * MB / F == a) dma(c + R, j, sc, f1);
        }
#pragma unroll
        for (int b = 0; b < 4; b++) mfma(av[st][a], bv[st][b], acc[a][b]);
        if (NBW == 5) {
          if (TR) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc5[a]) : "v"(bv[st][NBW - 1]), "v"(av[st][a]));
          else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc5[a]) : "v"(av[st][a]), "v"(bv[st][NBW - 1]));
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  } else {
    u32x4 av[2][2][MB], bv[2][2][4];      // [chunk parity][kb]
    constexpr int NM = 8 * MB, T = 2 * (MB + 4);      // MFMAs and operand reads of a chunk
#pragma unroll
    for (int j = 0; j < PW; j++) dma(c0 + R - 1, j, R - 1, behind(c0 + R - 1));
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((R - 1) * PW) : "memory");
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int kb = 0; kb < 2; kb++) {
#pragma unroll
      for (int x = 0; x < MB; x++) av[0][kb][x] = As[(kb * 4 + x) * 64];
#pragma unroll
      for (int x = 0; x < 4; x++) bv[0][kb][x] = Bs[(x * 2 + kb) * 64];
    }
    int sc = 0;                           // stage of chunk c
    auto chunk = [&](int c, auto parity) {
      constexpr int p = decltype(parity)::value;
      const int sn = sc + 1 == R ? 0 : sc + 1, base = sn * (BUF / 16), far = behind(c + R);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int m = 0; m < NM; m++) {
        const int kb = m / (4 * MB), a = m / 4 % MB, b = m % 4;
        if (m == 1) {      // chunk c + 1 has landed for every wave, chunk c is read out by every wave
          asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((R - 2) * PW) : "memory");
          __builtin_amdgcn_s_barrier();
        }
        mfma(av[p][kb][a], bv[p][kb][b], acc[a][b]);
        __builtin_amdgcn_sched_barrier(0);
        if (m > 0) {
#pragma unroll
          for (int q = 0; q < T; q++)
            if (1 + q * (NM - 4) / T == m) {
              const int k = q / (MB + 4), r = q % (MB + 4);
              if (r < 4) bv[1 - p][k][r] = Bs[base + (r * 2 + k) * 64];
              else av[1 - p][k][r - 4] = As[base + (k * 4 + r - 4) * 64];
            }
#pragma unroll
          for (int j = 0; j < PW; j++)
            if (2 + j * (NM - 2) / PW == m) dma(c + R, j, sc, far);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      sc = sn;
    };
    for (int c = c0; c < c1; c += 2) {
      chunk(c, std::integral_constant<int, 0>());
      if (c + 1 < c1) chunk(c + 1, std::integral_constant<int, 1>());
    }
  }
  // all loads into LDS are done; the last assembly MFMAs' results may be read
  if constexpr (NBW == 5)
    asm volatile("s_waitcnt vmcnt(0)\n\ts_nop 15\n\ts_nop 15"
                 : "+v"(acc5[0]), "+v"(acc5[1]), "+v"(acc5[2]), "+v"(acc5[3])::"memory");
  else
    asm volatile("s_waitcnt vmcnt(0)\n\ts_nop 15\n\ts_nop 15" ::: "memory");
  const int wrow0 = (blk0 + wm * MB) * 32;
  if ((wrow0 >> 7) >= (M + 127) >> 7) return;
  if constexpr (EPI == EPI_QKV || EPI == EPI_QKV8) {
    // every use reads its own element: the compiler otherwise keeps copies of whole 16-register
    // accumulators in vector registers and spills
    auto val = [&](int a, int b, int i) {
      if (MB == 2) return acc[a][b][i];
      float x;
      asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(x) : "a"(acc[a][b][i]));
      return x;
    };
    if (strip0 + wn * 4 < NB) qkv_head<EPI == EPI_QKV8, MB>(val, qkv, wrow0, M, (strip0 >> 2) + wn, lane);
    return;
  }
  float* Cp = (float*)Cv + (size_t)slice * M * N;
  if constexpr (EPI == EPI_ADD) {
    // C += product, one 32 x 32 block after the other; the addends are requested two blocks ahead
    if (wrow0 >= M) return;
    float old[3][16];
    const int last = M - 1 - wrow0, rsub = (lane >> 5) * 4;
    const int first = strip0 + wn * NBW;
    auto base = [&](int b) { return Cp + (size_t)wrow0 * N + min(first + b, NB - 1) * 32; };
    auto off = [&](int a, int i) { return (unsigned)(min(a * 32 + (i >> 2) * 8 + rsub + (i & 3), last) * N + (lane & 31)); };
    auto fetch = [&](int t) {
#pragma unroll
      for (int i = 0; i < 16; i++) old[t % 3][i] = base(t % NBW)[off(t / NBW, i)];
    };
    fetch(0);
    fetch(1);
#pragma unroll
    for (int t = 0; t < MB * NBW; t++) {
      const int a = t / NBW, b = t % NBW;
      if (t + 2 < MB * NBW) fetch(t + 2);
      __builtin_amdgcn_sched_barrier(0);
      if (first + b < NB) {
#pragma unroll
        for (int i = 0; i < 16; i++) {
          const float v = old[t % 3][i] + (b < 4 ? acc[a][b & 3][i] : acc5[a][i]);
          if (a * 32 + (i >> 2) * 8 + rsub + (i & 3) <= last) __builtin_nontemporal_store(v, &base(b)[off(a, i)]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    return;
  }
#pragma unroll
  for (int a = 0; a < MB; a++) {
    const int row0 = wrow0 + a * 32, row = row0 + (lane & 31);
#pragma unroll
    for (int b = 0; b < NBW; b++) {
      const int nb = strip0 + wn * NBW + b;
      if (nb >= NB) continue;
      auto val = [&](int i) { return b < 4 ? acc[a][b & 3][i] : acc5[a][i]; };
      if constexpr (EPI == EPI_SWIGLU) {
        swiglu_block(val, (bf16_t*)Cv, row, M, nb, lane, N >> 1);
      } else if constexpr (EPI == EPI_LSE) {
        lse_block(val, (float2*)Cv, zt, tgt, row, M, nb, NB, lane, scale_c);
      } else {
        const int col = nb * 32 + (lane & 31);
#pragma unroll
        for (int i = 0; i < 16; i++) {
          const int r = row0 + (i >> 2) * 8 + (lane >> 5) * 4 + (i & 3);
          if (r < M) __builtin_nontemporal_store(val(i), &Cp[(size_t)r * N + col]);
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);      // one row block's values in flight at a time
  }
}

constexpr int kLdsBytes = 160 * 1024;     // of a CU
// More than 64 KB of dynamic LDS need an opt-in, once per kernel and device.
static void set_lds_limit(std::atomic<uint64_t>& done, const void* kernel, int bytes) {
  int dev = 0;
  (void)hipGetDevice(&dev);
  const uint64_t bit = 1ull << (dev & 63);
  if (done.load(std::memory_order_acquire) & bit) return;
  (void)hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  done.fetch_or(bit, std::memory_order_release);
}

// Stages of the ring, and the grid of a launch.
static int dma_stages(int mb, int epilogue, const dim3& grid, int chunks_per_split) {
  if (mb == 4) return 4;
  return epilogue != EPI_QKV && epilogue != EPI_QKV8 && grid.x * grid.y * grid.z <= 256 && chunks_per_split >= 48 ? 4 : 3;
}
static dim3 dma_grid(int mb, int nbw, int M, int N, int splits) {
  return dim3((N / 32 + 2 * nbw - 1) / (2 * nbw), (M + 64 * mb - 1) / (64 * mb), splits);
}

void debug_many_row_loads(int M, int N, int K, int mb, int nbw, int splits, int epilogue, int64_t* out) {
  const int cps = (K / 32 + splits - 1) / splits, tiles128 = (M + 127) / 128;
  const dim3 grid = dma_grid(mb, nbw, M, N, splits);
  const int stages = dma_stages(mb, epilogue, grid, cps);
  int64_t far_rows = 0, far_weights = 0;
  for (int z = 0; z < splits; z++)
    for (unsigned y = 0; y < grid.y; y++)
      for (unsigned x = 0; x < grid.x; x++) {
        const int mts = std::min(tiles128 - (int)y * mb / 2, mb / 2), c1 = std::min((z + 1) * cps, K / 32);
        const ManyRowLoads at{c1, N / 32, (int)x * 2 * nbw, mts > 1 ? (unsigned)K * 256u : 0u};
        for (int c = z * cps; c < c1 + stages; c++)
          for (int j = 0; j < mb + nbw; j++)
            for (int wave = 0; wave < 4; wave++) {
              if (j < mb) far_rows = std::max(far_rows, at.rows(c, j >> 1, j & 1, wave) + 1024 - (int64_t)mts * K * 256);
              else far_weights = std::max(far_weights, at.weights(c, j - mb, wave) + 1024 - (int64_t)N * K * 2);
            }
      }
  out[0] = stages;
  out[1] = far_rows;
  out[2] = far_weights;
}

template <int EPI, int MB, int NBW>
static void launch_dma(hipStream_t s, const bf16_t* A, const bf16_t* Wp, void* C, int M, int N, int K, int splits,
                       const int32_t* tgt, float* zt, float scale_c, const QkvArgs& q) {
  const int cps = (K / 32 + splits - 1) / splits;
  const dim3 grid = dma_grid(MB, NBW, M, N, splits);
  static std::atomic<uint64_t> done[2];
  auto go = [&](auto kernel, int stages) {
    const int lds = stages * (4 * MB + 4 * NBW) * 1024;
    set_lds_limit(done[stages - 3], (const void*)kernel, lds);
    kernel<<<grid, 256, lds, s>>>(A, Wp, C, M, N, K, cps, tgt, zt, scale_c, q);
  };
  if constexpr (MB == 4) {
    go(gemm_dma_kernel<EPI, 4, NBW, 4>, 4);
  } else {
    if constexpr (EPI != EPI_QKV && EPI != EPI_QKV8) {
      if (dma_stages(MB, EPI, grid, cps) == 4) return go(gemm_dma_kernel<EPI, 2, 4, 4>, 4);
    }
    go(gemm_dma_kernel<EPI, 2, 4, 3>, 3);
  }
}

// =============================================================================================
// GEMM for decode batches of 33 to 128 rows and, where the estimate says so, fewer: tile 64 * RB rows
// (RB = 1 or 2 16-row blocks per wave) x 16 * CB columns.  What bounds these products is what one CU can
// fetch: about 27 GB/s of weights from HBM and 125 GB/s of activations, which every workgroup needs
// whole, from L2.  So the work is cut for 256 equal workgroups (CB = 2, 4, 5 or 6, times K-slices: 80
// columns of the 4B gate-up make 244, where 128-column tiles leave 104 CUs idle), and both operands
// stream straight into an LDS ring of NST stages of SK k, NST - 1 ahead, with one barrier per stage and
// no staging registers.  A block is 16 rows (columns) x 32 k in operand order, gathered from the 32-row
// layout by the lanes' offsets.  The product is formed transposed: four consecutive columns of a row
// per lane, stored as 16 bytes; SwiGLU needs one swap of lane halves.
// Rows are whole-wave work with no sum across waves: a row's bits do not depend on its place.
// us at 128 / 64 rows, the 128-column kernel -> this: gate-up N = 19456 K = 2560 28.8 -> 26.0 / 23.4 -> 19.0,
// down N = 2560 K = 9728 17.9 -> 15.9 / 14.1 -> 11.9, O N = 2560 K = 4096 9.9 -> 8.5 / 7.9 -> 6.7, QKV
// N = 6144 K = 2560 11.7 -> 10.7 / 8.6 -> 8.4; 0.6B shape: gate-up 11.3 -> 7.2 / 7.5 -> 5.7, down 7.0 -> 4.4 /
// 4.8 -> 3.6.  NT (up to 64 rows, weights of 24 MB and more): weights past the caches, at 16 rows 8B gate-up N = 24576
// K = 4096 34.3 -> 32.2 us (6.3 TB/s), down N = 4096 K = 12288 17.8 -> 17.1, O 8.0 -> 7.6, 4B QKV 7.5 -> 7.2, gate-up 18.3 ->
// 17.9; at 96 rows 0 to 2 %.  Deeper rings gain nothing; leaving out the loads behind the slice with a branch costs
// 10 % (the loop falls apart into blocks).
// =============================================================================================
// UNDIV (SwiGLU): the rows of A are still to be divided by their rms, ssq holds their sums of squares.  The epilogue adds up K / 64
// of them per lane, 0.6 to 1 us (8B gate-up in a pass of 6 / 16 rows 33.5 / 34.8 us, 6.0 / 5.8 TB/s; 4B at 37 rows 18.8 ->
// 19.8, hidden 1024 at 64 rows 6.2 -> 6.8).  A choice at compile time: tested at run time it had grown the plain form from
// 12.5 to 15 KB of code.
template <int EPI, int RB, int CB, int SK, int NST, bool NT, bool UNDIV>
__global__ __launch_bounds__(256) void gemm_decode_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ Wp,
                                                       void* __restrict__ Cv, int M, int N, int K, int splits,
                                                       int stages_per_split, const float* __restrict__ ssq, float eps) {
  constexpr int KB = SK / 32;                    // 32-k steps of a stage
  constexpr int NA = 4 * RB * KB, NW = CB * KB;  // blocks
  constexpr int PW = (NA + NW) / 4;
  static_assert((NST - 2) * PW <= 63 && NST <= 7, "wait counter");
  static_assert((NA + NW) % 4 == 0, "even");
  constexpr int BUF = (NA + NW) * 1024;
  extern __shared__ u32x4 smem[];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  // Slices of a tile are neighbours, except four long ones: dealt round-robin to the 8 XCDs they would put every other
  // tile of a slice on an XCD (N = 4096 K = 4096 at 16 rows, 64 columns: 9.4 us; K = 12288 21.0).  There an XCD takes a
  // contiguous range of tiles of one slice (7.9, 17.9; N = 6144 K = 4096 10.4 -> 10.2).  Other counts, slices under
  // 512 k and more than 64 rows are better off, or no worse, the plain way (N = 4096 K = 1024: 3.7 against 4.3; N = 6144
  // K = 2560 at 128 rows 10.7 against 11.0).
  int tile, split;
  if constexpr (EPI == EPI_SWIGLU) {      // one slice
    tile = blockIdx.x;
    split = 0;
  } else if (RB == 1 && splits == 4 && stages_per_split * SK >= 512) {
    const int tiles = gridDim.x / 4, base = gridDim.x >> 3, rem = gridDim.x & 7, x = blockIdx.x & 7;
    const int v = x * base + min(x, rem) + (blockIdx.x >> 3);
    split = __builtin_amdgcn_readfirstlane(v / tiles);
    tile = __builtin_amdgcn_readfirstlane(v - split * tiles);
  } else {
    tile = blockIdx.x / splits;
    split = blockIdx.x - tile * splits;
  }
  const int NB = N >> 5, N16 = N >> 4, nst = K / SK;
  const int s0 = split * stages_per_split, s1 = EPI == EPI_SWIGLU ? nst : min(s0 + stages_per_split, nst);
  const int r16 = (M + 15) >> 4;      // 16-row blocks in use: the others are not fetched
  const u32x4 ra = buffer_rsrc(A, (unsigned)K * 256u), rw = buffer_rsrc(Wp, (unsigned)N * (unsigned)K * 2u);
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void*)smem;
  const int lp = ((lane & 15) + (((lane >> 4) & 1) << 5)) << 4;
  const int lw = ((lane >> 5) << 10) + lp, la = ((lane >> 5) << 12) + lp;
  // piece j of this wave of stage s: block id j * 4 + wave, weight blocks first; stages behind the slice
  // and row blocks without rows are asked for behind the buffer's end: no memory traffic (gate-up of the 4B shape at 1 to
  // 48 rows 18.8 -> 18.1 us, 80 rows 25.5 -> 24.5; 8B QKV at 80 rows 13.4 -> 12.1), and the count of loads stays the same
  auto dma = [&](int s, int j) {
    const int sl = min(s, s1 - 1), id = j * 4 + wave;
    const unsigned dst = lds0 + (unsigned)((s - s0) % NST) * BUF + (unsigned)id * 1024u;
    if (id < NW) {
      const int t = sl * KB + id / CB, c16 = min(tile * CB + id % CB, N16 - 1);   // columns past the end: dropped
      load_to_lds<NT>(dst, s < s1 ? lw : 0x7fff0000, rw,
                  ((unsigned)(t >> 1) * NB + (c16 >> 1)) * 4096u + (t & 1) * 2048u + (c16 & 1) * 256u);
    } else {
      const int x = id - NW, r = x % (4 * RB), t = sl * KB + x / (4 * RB);
      load_to_lds(dst, s < s1 && r < r16 ? la : 0x7fff0000, ra, (unsigned)t * 8192u + (r >> 1) * 1024u + (r & 1) * 256u);
    }
  };
  f32x4 acc[CB][RB];
#pragma unroll
  for (int c = 0; c < CB; c++)
#pragma unroll
    for (int r = 0; r < RB; r++) acc[c][r] = (f32x4){0.f, 0.f, 0.f, 0.f};
  // the sums of squares behind the ring; the ring's loads are younger, so its first wait covers these
  if (UNDIV) {
    const int ss_bytes = r16 * (K >> 4) * 64;
    const u32x4 rs = buffer_rsrc(ssq, (unsigned)ss_bytes);
    for (int p = wave; p * 1024 < ss_bytes; p += 4) load_to_lds(lds0 + NST * BUF + p * 1024, lane * 16, rs, (unsigned)p * 1024u);
  }
#pragma unroll
  for (int p = 0; p < NST - 1; p++)
#pragma unroll
    for (int j = 0; j < PW; j++) dma(s0 + p, j);
  int buf = 0;
  for (int s = s0; s < s1; s++) {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NST - 2) * PW) : "memory");
    __builtin_amdgcn_s_barrier();
    const u32x4* B = smem + buf * (BUF / 16) + lane;
    buf = buf + 1 == NST ? 0 : buf + 1;
    u32x4 w[2][CB], a[2][RB];
    auto rd = [&](int k) {
#pragma unroll
      for (int c = 0; c < CB; c++) w[k & 1][c] = B[(k * CB + c) * 64];
#pragma unroll
      for (int r = 0; r < RB; r++) a[k & 1][r] = B[(NW + k * 4 * RB + wave * RB + r) * 64];
    };
    rd(0);
#pragma unroll
    for (int k = 0; k < KB; k++) {
      if (k + 1 < KB) rd(k + 1);
#pragma unroll
      for (int j = 0; j < PW; j++)
        if (j * KB / PW == k ) dma(s + NST - 1, j);
#pragma unroll
      for (int c = 0; c < CB; c++)
#pragma unroll
        for (int r = 0; r < RB; r++)
          acc[c][r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[k & 1][c]),
                                                              __builtin_bit_cast(bf16x8, a[k & 1][r]), acc[c][r], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
  for (int r = 0; r < RB; r++) {
    const int row = (wave * RB + r) * 16 + (lane & 15);
    float inv = 1.0f;
    if (UNDIV) {       // the row's norm: every lane group of 16 sums every fourth partial sum
      const float* sq = (const float*)(smem + NST * (BUF / 16)) + min(row, r16 * 16 - 1);
      float t = strided_sum(sq, lane >> 4, 4, K >> 4, r16 * 16);
      t += __shfl_xor(t, 16, 64);
      t += __shfl_xor(t, 32, 64);
      inv = 1.0f / sqrtf(t / (float)K + eps);
    }
#pragma unroll
    for (int c = 0; c < CB; c++) {
      const int c16 = tile * CB + c;
      if (c16 >= N16) continue;
      f32x4 v = acc[c][r];
      if (EPI == EPI_SWIGLU) {
        if (UNDIV) v *= inv;
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
}

// LDS of a workgroup: the ring and, with the rows' sums of squares, those of `scaled` rows
static int decode_gemm_lds(int M, int K, int cb, bool scaled) {
  const int rb = M <= 64 ? 1 : 2, sk = cb == 5 ? 128 : 64, nst = cb == 5 ? 3 : 4;
  return nst * (4 * rb + cb) * (sk / 32) * 1024 + (scaled ? ((M + 15) / 16 * (K / 16) * 64 + 1023) / 1024 * 1024 : 0);
}
template <int EPI, int CB, bool UNDIV>
static void launch_decode_gemm(hipStream_t s, const bf16_t* A, const bf16_t* Wp, void* C, int M, int N, int K, int splits,
                               const float* ssq, float eps) {
  constexpr int SK = CB == 5 ? 128 : 64, NST = CB == 5 ? 3 : 4;   // CB = 5: whole rounds of 4 waves need 128 k
  const int rb = M <= 64 ? 1 : 2, lds = decode_gemm_lds(M, K, CB, UNDIV);
  const bool nt = rb == 1 && streams_weights(N, K);
  static std::atomic<uint64_t> done[3];
  auto go = [&](auto kernel) {
    set_lds_limit(done[nt ? 2 : rb - 1], (const void*)kernel, kLdsBytes);
    const int sps = (K / SK + splits - 1) / splits;
    kernel<<<(N / 16 + CB - 1) / CB * splits, 256, lds, s>>>(A, Wp, C, M, N, K, splits, sps, ssq, eps);
  };
  if (nt) go(gemm_decode_kernel<EPI, 1, CB, SK, NST, true, UNDIV>);
  else if (rb == 1) go(gemm_decode_kernel<EPI, 1, CB, SK, NST, false, UNDIV>);
  else go(gemm_decode_kernel<EPI, 2, CB, SK, NST, false, UNDIV>);
}

// =============================================================================================
// O and down of few rows, with the residual add and the norm behind them: h += A * W^T, out = bf16(h * g) in A-tile
// layout, not yet divided by the row's rms, and per 16 columns the row's sum of squares, ssq[N / 16][rows in
// use rounded up to 16].  The consumer (QKV's norm / RoPE kernel, gate-up's epilogue) divides: a row's factor commutes with the
// product, and bf16 rounds h g and h g / rms alike.  The separate norm (4 to 6 us: a launch and a chain of memory
// round trips for a few KB per row) and the fp32 partial sums between the two are gone.
// Tile 16 RB rows x 16 CB columns, as narrow as gives most CUs a workgroup without slicing K over workgroups; the
// workgroup's four waves take every fourth 32-k step, operands straight to registers, U steps in flight, and one wave per
// 16 x 16 block adds the four sums in ascending order: a row's bits depend on neither the tile nor the row count.  (Eight waves:
// 0 to 1 us slower.)  Bound by the weights' stream (16 rows) and by what a CU fetches (about
// 50 GB/s of both operands): more rows re-read the weights in every row tile, so it is taken where its estimate beats
// the sliced product and the norm (plan_residual).
// us, sliced product + norm -> this: N = 1024 K = 2048 at 1 / 64 rows 6.8 -> 4.4 / 7.7 -> 4.0, K = 3072 at 64 8.2 -> 5.1;
// N = 2560 K = 4096 at 16 / 64 11.9 -> 7.2 / 12.5 -> 10.9, K = 9728 at 16 15.7 -> 14.0; N = 4096 K = 4096 at 16 / 64
// 13.4 -> 8.3 / 14.8 -> 11.6, K = 12288 at 16 24.0 -> 18.9.
// =============================================================================================
template <int RB, int CB, int U, bool NT>
__global__ __launch_bounds__(256) void gemm_residual_kernel(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ Wp, float* __restrict__ h, const bf16_t* __restrict__ g,
    bf16_t* __restrict__ out, float* __restrict__ ssq, int M, int N, int K, int row_tiles) {
  constexpr int NW = 4, NBLK = RB * CB, OWN = (NBLK + NW - 1) / NW;      // 16 x 16 blocks, and those that a wave finishes
  __shared__ f32x4 red[NW][NBLK][64];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int NB = N >> 5, N16 = N >> 4, steps = K >> 5, r16 = (M + 15) >> 4;
  // the row tiles of a column tile follow each other on one XCD, whose L2 then has the weights
  int ct = blockIdx.x, rt = 0;
  if (row_tiles > 1) {
    const int y = blockIdx.x >> 3;
    rt = y % row_tiles;
    ct = y / row_tiles * 8 + (blockIdx.x & 7);
  }
  if (ct * CB >= N16) return;
  const auto ra = __builtin_amdgcn_make_buffer_rsrc((void*)A, 0, ((M + 127) >> 7) * K * 256, 0x00027000);
  const auto rw = __builtin_amdgcn_make_buffer_rsrc((void*)Wp, 0, (int)((unsigned)N * (unsigned)K * 2u), 0x00027000);
  const int lp = ((lane & 15) + (((lane >> 4) & 1) << 5)) << 4;
  const int lw = ((lane >> 5) << 10) + lp, la = ((lane >> 5) << 12) + lp;
  f32x4 acc[CB][RB];
#pragma unroll
  for (int c = 0; c < CB; c++)
#pragma unroll
    for (int r = 0; r < RB; r++) acc[c][r] = (f32x4){0.f, 0.f, 0.f, 0.f};
  u32x4 w[U][CB], a[U][RB];
  auto fetch = [&](int u, int t) {      // steps behind the end and row blocks without rows: behind the buffer, zeros
    const bool in = t < steps;
#pragma unroll
    for (int c = 0; c < CB; c++) {
      const int c16 = ct * CB + c;
      const int so = ((t >> 1) * NB + (c16 >> 1)) * 4096 + (t & 1) * 2048 + (c16 & 1) * 256;
      w[u][c] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                              rw, in && c16 < N16 ? lw : 0x7fff0000, in && c16 < N16 ? so : 0, NT ? 2 : 0));
    }
#pragma unroll
    for (int r = 0; r < RB; r++) {
      const int x = rt * RB + r;
      const int so = (x >> 3) * K * 256 + t * 8192 + (x >> 1 & 3) * 1024 + (x & 1) * 256;
      a[u][r] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                              ra, in && x < r16 ? la : 0x7fff0000, in && x < r16 ? so : 0, 0));
    }
  };
#pragma unroll
  for (int u = 0; u < U; u++) fetch(u, wave + u * NW);
  f32x4 old[OWN];
  uint2 gw[OWN];
#pragma unroll
  for (int k = 0; k < OWN; k++) {
    const int b = k * NW + wave, row = (rt * RB + b % RB) * 16 + (lane & 15), col = (ct * CB + b / RB) * 16 + 4 * (lane >> 4);
    old[k] = (f32x4){0.f, 0.f, 0.f, 0.f};
    gw[k] = make_uint2(0u, 0u);
    if (b < NBLK && row < M && col < N) {
      old[k] = *(const f32x4*)(h + (size_t)row * N + col);
      gw[k] = *(const uint2*)(g + col);
    }
  }
  for (int t = wave; t < steps; t += NW * U) {
#pragma unroll
    for (int u = 0; u < U; u++) {
#pragma unroll
      for (int c = 0; c < CB; c++)
#pragma unroll
        for (int r = 0; r < RB; r++)
          acc[c][r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[u][c]),
                                                              __builtin_bit_cast(bf16x8, a[u][r]), acc[c][r], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      fetch(u, t + (u + U) * NW);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int c = 0; c < CB; c++)
#pragma unroll
    for (int r = 0; r < RB; r++) red[wave][c * RB + r][lane] = acc[c][r];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < OWN; k++) {
    const int b = k * NW + wave;
    if (b >= NBLK) break;
    const int row = (rt * RB + b % RB) * 16 + (lane & 15), c16 = ct * CB + b / RB, col = c16 * 16 + 4 * (lane >> 4);
    f32x4 v = red[0][b][lane];
#pragma unroll
    for (int x = 1; x < NW; x++) v += red[x][b][lane];
    v += old[k];
    float ss = (v[0] * v[0] + v[1] * v[1]) + (v[2] * v[2] + v[3] * v[3]);
    ss += __shfl_xor(ss, 16, 64);
    ss += __shfl_xor(ss, 32, 64);
    if (row >= M || c16 >= N16) continue;
    *(f32x4*)(h + (size_t)row * N + col) = v;
    const uint32_t y0 = f2bf(v[0] * bf2f((bf16_t)(gw[k].x & 0xffff))), y1 = f2bf(v[1] * bf2f((bf16_t)(gw[k].x >> 16)));
    const uint32_t y2 = f2bf(v[2] * bf2f((bf16_t)(gw[k].y & 0xffff))), y3 = f2bf(v[3] * bf2f((bf16_t)(gw[k].y >> 16)));
    *(uint2*)(out + atile_off(row, col, N)) = make_uint2(y0 | (y1 << 16), y2 | (y3 << 16));
    if (lane < 16) ssq[(size_t)c16 * (r16 * 16) + row] = ss;
  }
}

// Tile of the product with residual add and norm, and its estimate in us: per round of 256 workgroups 1.28, 1.75 or
// 2.1 us per 1000 k for 16 x 16, 16 x 32 and 32 x 32 (what the workgroup's operands take), plus the launch and what the
// consumer takes to add up the sums of squares.  Fitted on six products of hidden 1024 to 4096 at 1 to 128 rows.
// More rows: the same tile, its time (without the consumer) by rounds, by what the row tiles re-read of the weights and by the
// residual stream's traffic; fitted to 0.65 us on 18 shapes of hidden 512 to 5120 at 131 to 512 rows (see plan_pass).
// rb = 0: not for this size.
ResidualPlan plan_residual(int M, int N, int K) {
  ResidualPlan best{0, 0, 1e30};
  // 31-bit offsets into the weights and into the row tiles
  if (M > kResidualRows || (size_t)N * K * 2 >= 0x7fff0000ull || (size_t)((M + 127) / 128) * K * 256 >= 0x7fff0000ull) return best;
  const struct { int rb, cb; double launch, per_k; } tiles[] = {{1, 1, 3.0, 1.28e-3}, {1, 2, 3.0, 1.75e-3}, {2, 2, 3.1, 2.1e-3}};
  for (const auto& t : tiles) {
    const int wgs = (M + 16 * t.rb - 1) / (16 * t.rb) * ((N / 16 + t.cb - 1) / t.cb);
    const double cost = t.launch + (wgs + 255) / 256 * (K * t.per_k);
    if (cost < best.cost) best = ResidualPlan{t.rb, t.cb, cost};
  }
  if (M > 128) {
    const int wgs = (M + 16 * best.rb - 1) / (16 * best.rb) * ((N / 16 + best.cb - 1) / best.cb);
    best.cost = 2.5 + K * ((best.rb == 2 ? 0.8e-3 : 0.45e-3) * ((wgs + 255) / 256) + 0.68e-3 * wgs / 256) + 3.7e-6 * M * N;
  }
  return best;
}
bool gate_up_takes_scale(const GemmPlan& plan, int M, int K) {
  return plan.kind == GEMM_TILE128 || (plan.kind == GEMM_DECODE && decode_gemm_lds(M, K, plan.width, true) <= kLdsBytes);
}

void launch_gemm_residual(hipStream_t s, const bf16_t* A, const bf16_t* Wp, float* h, const bf16_t* g, bf16_t* out, float* ssq,
                          int M, int N, int K, const ResidualPlan& plan) {
  if (M <= 0) return;
  const int rt = (M + 16 * plan.rb - 1) / (16 * plan.rb), ct = (N / 16 + plan.cb - 1) / plan.cb;
  const int grid = rt == 1 ? ct : (ct + 7) / 8 * 8 * rt;
  const bool nt = rt == 1 && streams_weights(N, K);
  auto go = [&](auto kernel) { kernel<<<grid, 256, 0, s>>>(A, Wp, h, g, out, ssq, M, N, K, rt); };
  if (plan.cb == 1 && nt) go(gemm_residual_kernel<1, 1, 8, true>);
  else if (plan.cb == 1) go(gemm_residual_kernel<1, 1, 8, false>);
  else if (plan.rb == 1 && nt) go(gemm_residual_kernel<1, 2, 6, true>);
  else if (plan.rb == 1) go(gemm_residual_kernel<1, 2, 6, false>);
  else if (nt) go(gemm_residual_kernel<2, 2, 4, true>);
  else go(gemm_residual_kernel<2, 2, 4, false>);
}

template <int EPI, bool UNDIV = false>
static void gemm_launch(hipStream_t s, const bf16_t* A, const bf16_t* Wp, void* C, int M, int N, int K, int splits, int cps,
                        float* zt, float scale_c) {
  const dim3 grid((N + 127) / 128, (M + 127) / 128, splits);
  auto go = [&](auto kernel) { kernel<<<grid, 256, 0, s>>>(A, Wp, C, M, N, K, cps, nullptr, zt, scale_c); };
  const bool nt = streams_weights(N, K);
  if (M <= 32 && nt) go(gemm_mfma_kernel<EPI, 1, true, UNDIV>);      // row blocks in use (one row tile when < 4)
  else if (M <= 32) go(gemm_mfma_kernel<EPI, 1, false, UNDIV>);
  else if (M <= 64 && nt) go(gemm_mfma_kernel<EPI, 2, true, UNDIV>);
  else if (M <= 64) go(gemm_mfma_kernel<EPI, 2, false, UNDIV>);
  else go(gemm_mfma_kernel<EPI, 4, false, UNDIV>);
}

// Which kernel and how many K-slices: the cheapest by estimate (us), over at most kMaxSplits slices of
// at least 256 k.  Further partial sums cost their stores and their reading at 5 TB/s.
// At most 128 rows: per round of 256 workgroups the time of a workgroup's weight bytes and of its activation bytes,
// plus the launch.  Up to 64 rows: decode kernel 27 and 113 GB/s (the 16-row blocks in use), 2.2 us, and with 32 columns
// no less than 0.25 us per 64 k (the ring then holds too few bytes to cover the latency); 128-column kernel 29 and 103
// GB/s, 2.7 us.  Above: 27 and 125 GB/s (128 rows) for both, 2.2 and 3.2 us.  The 128-column kernel fetches the 32-row
// blocks in use and stays the better one where its 128 columns times slices make whole rounds (8B down at N = 4096
// K = 12288, 48 rows: 18.7 against 19.5 us with 96 columns).  Fitted on 20 products of hidden 1024 to 4096 at 1 to 128
// rows: with the reading of its partial sums the plan's product is 0.9 % above the best plan's on average, 10 % at most.
// More rows: a round is 256 workgroups, one per CU.  256-row tiles cost per 32-k chunk 0.43 us with most
// CUs idle to 0.73 us with all of them busy (320 columns: 1.25 times that) and 4 to 16 us per round to
// store a tile; 128 x 256 tiles 0.46 us per chunk and 5 us per round (two share a CU, at the speed of one
// after the other); 128 x 128 tiles 0.62 us per 64-k chunk and round, 0.59 us from the second round on
// (several to a CU).  Fitted on N = 2048 to 6144, K = 640 to 9728, 64 to 1280 tiles; e.g. 8192 x 2560 x
// 9728: 320 columns make one full round of 256 tiles (289 us) where 256 columns make two (398 us).
// The 128 x 256 tiles' loop has become faster since (0.40 us per chunk); with the old constants the plan's product is still 1.1 %
// above the best plan's on average (209 products of hidden 512 to 4096 at 131 to 4096 rows, refitted 0.6 %).
GemmPlan plan_gemm(int M, int N, int K, int epilogue, size_t part_rows) {
  const bool can_split = epilogue == EPI_STORE;
  int most = can_split ? (int)std::min<size_t>(kMaxSplits, std::max<size_t>(1, part_rows / (size_t)std::max(M, 1))) : 1;
  most = std::min(most, std::max(1, K / 256));
  const bool wide = (size_t)N * K * 2 >= 0x7fff0000ull;      // beyond a buffer descriptor's signed offsets
  const double part = (double)M * N * 4.0 / 5.0e6;           // one partial sum, stored or read
  const int tiles = ((N + 127) / 128) * ((M + 127) / 128), nch = K / 64;
  GemmPlan best{GEMM_TILE128, 0, 1, 1e30};
  auto offer = [&](int kind, int width, int splits, double cost) {
    if (cost < best.cost) best = GemmPlan{kind, width, splits, cost};
  };
  if (M <= 128) {
    const double arow = (M <= 32 ? 32 : M <= 64 ? 64 : 128) * 2.0, adec = M <= 64 ? (M + 15) / 16 * 32.0 : 256.0;
    const bool few = M <= 64;
    for (int sp = 1; sp <= most; sp++) {
      const int cps = (nch + sp - 1) / sp, r = (tiles * sp + 255) / 256;
      offer(GEMM_TILE128, 0, sp, (few ? 2.7 : 3.2) + r * cps * 64 * (256 / (few ? 29.0e3 : 27.0e3) + arow / (few ? 103.0e3 : 125.0e3)) +
                                     (2 * sp - 1) * part);
      if (wide || (epilogue != EPI_STORE && epilogue != EPI_SWIGLU)) continue;
      for (int cb : {2, 4, 5, 6}) {
        const int sk = cb == 5 ? 128 : 64;
        if (K % sk != 0) continue;
        const int k = (K / sk + sp - 1) / sp * sk, rd = ((N / 16 + cb - 1) / cb * sp + 255) / 256;
        const double t = std::max(k * (32 * cb / 27.0e3 + adec / (few ? 113.0e3 : 125.0e3)), cb == 2 && few ? k / 64 * 0.25 : 0.0);
        offer(GEMM_DECODE, cb, sp, 2.2 + rd * t + (2 * sp - 1) * part);
      }
    }
    if (best.kind == GEMM_DECODE) {     // no empty slices
      const int st = K / (best.width == 5 ? 128 : 64), sps = (st + best.splits - 1) / best.splits;
      best.splits = (st + sps - 1) / sps;
    }
    return best;
  }
  int s = 1;
  if (M <= 1024 && tiles < 240) s = std::max(1, std::min((240 + tiles / 2) / tiles, most));
  const int rounds = (tiles * s + 255) / 256;
  offer(GEMM_TILE128, 0, s, 7.0 + rounds * (rounds > 1 ? 0.59 : 0.62) * ((nch + s - 1) / s) + (s - 1) * part);
  if (wide) return best;
  for (int nbw = 4; nbw <= (epilogue == EPI_STORE || epilogue == EPI_SWIGLU ? 5 : 4); nbw++)
    for (int sp = 1; sp <= most; sp++) {
      const int t = ((N / 32 + 2 * nbw - 1) / (2 * nbw)) * ((M + 255) / 256) * sp, r = (t + 255) / 256;
      const double fill = t / (256.0 * r), w = nbw / 4.0;
      const int cps = (K / 32 + sp - 1) / sp;
      offer(GEMM_TILE256, nbw, (K / 32 + cps - 1) / cps,
            3.0 + r * (cps * w * (0.43 + 0.30 * fill) + 4.0 + 10.0 * w * fill) + (sp - 1) * part);
    }
  if (epilogue != EPI_LSE)
    for (int sp = 1; sp <= most; sp++) {
      const int t = ((N / 32 + 7) / 8) * ((M + 127) / 128) * sp, cps = (K / 32 + sp - 1) / sp;
      const double r = t <= 512 ? (t + 255) / 256 : t / 256.0;
      offer(GEMM_WIDE128, 4, (K / 32 + cps - 1) / cps, 3.0 + r * (cps * 0.46 + 5.0) + (sp - 1) * part);
    }
  return best;
}

int launch_gemm_mfma(hipStream_t s, const bf16_t* A, const bf16_t* Wp, void* C, int M, int N, int K, int epilogue,
                     const GemmPlan& plan, const float* ssq, float eps) {
  if (M <= 0) return 0;
  const int width = plan.width, sp = plan.splits;
  const QkvArgs none{};
  if (plan.kind == GEMM_WIDE128) {
    if (epilogue == EPI_STORE) launch_dma<EPI_STORE, 2, 4>(s, A, Wp, C, M, N, K, sp, nullptr, nullptr, 0.f, none);
    else if (epilogue == EPI_ADD) launch_dma<EPI_ADD, 2, 4>(s, A, Wp, C, M, N, K, 1, nullptr, nullptr, 0.f, none);
    else launch_dma<EPI_SWIGLU, 2, 4>(s, A, Wp, C, M, N, K, 1, nullptr, nullptr, 0.f, none);
    return epilogue == EPI_ADD ? 0 : sp;
  }
  if (plan.kind == GEMM_TILE256) {
    if (epilogue == EPI_STORE && width == 4) launch_dma<EPI_STORE, 4, 4>(s, A, Wp, C, M, N, K, sp, nullptr, nullptr, 0.f, none);
    else if (epilogue == EPI_STORE) launch_dma<EPI_STORE, 4, 5>(s, A, Wp, C, M, N, K, sp, nullptr, nullptr, 0.f, none);
    else if (epilogue == EPI_ADD && width == 4) launch_dma<EPI_ADD, 4, 4>(s, A, Wp, C, M, N, K, 1, nullptr, nullptr, 0.f, none);
    else if (epilogue == EPI_ADD) launch_dma<EPI_ADD, 4, 5>(s, A, Wp, C, M, N, K, 1, nullptr, nullptr, 0.f, none);
    else if (width == 4) launch_dma<EPI_SWIGLU, 4, 4>(s, A, Wp, C, M, N, K, 1, nullptr, nullptr, 0.f, none);
    else launch_dma<EPI_SWIGLU, 4, 5>(s, A, Wp, C, M, N, K, 1, nullptr, nullptr, 0.f, none);
    return epilogue == EPI_ADD ? 0 : sp;
  }
  if (plan.kind == GEMM_DECODE) {
    auto go = [&](auto epi, auto undiv) {
      constexpr int E = decltype(epi)::value;
      constexpr bool U = decltype(undiv)::value;
      if (width == 2) launch_decode_gemm<E, 2, U>(s, A, Wp, C, M, N, K, sp, ssq, eps);
      else if (width == 4) launch_decode_gemm<E, 4, U>(s, A, Wp, C, M, N, K, sp, ssq, eps);
      else if (width == 5) launch_decode_gemm<E, 5, U>(s, A, Wp, C, M, N, K, sp, ssq, eps);
      else launch_decode_gemm<E, 6, U>(s, A, Wp, C, M, N, K, sp, ssq, eps);
    };
    if (epilogue == EPI_STORE) go(std::integral_constant<int, EPI_STORE>(), std::false_type());
    else if (!ssq) go(std::integral_constant<int, EPI_SWIGLU>(), std::false_type());
    else go(std::integral_constant<int, EPI_SWIGLU>(), std::true_type());
    return sp;
  }
  const int nchunks = K / 64;
  int splits = epilogue == EPI_SWIGLU ? 1 : std::max(1, std::min(sp, nchunks));
  const int cps = (nchunks + splits - 1) / splits;
  splits = (nchunks + cps - 1) / cps;
  if (epilogue == EPI_STORE) gemm_launch<EPI_STORE>(s, A, Wp, C, M, N, K, splits, cps, nullptr, 0.f);
  else if (!ssq) gemm_launch<EPI_SWIGLU>(s, A, Wp, C, M, N, K, splits, cps, nullptr, 0.f);
  else gemm_launch<EPI_SWIGLU, true>(s, A, Wp, C, M, N, K, splits, cps, const_cast<float*>(ssq), eps);
  return splits;
}

void launch_gemm_qkv(hipStream_t s, const bf16_t* A, const bf16_t* Wp, int M, int N, int K, bool kv_fp8,
                     const GemmPlan& plan, const QkvArgs& q) {
  if (M <= 0) return;
  if (plan.kind == GEMM_WIDE128) {
    if (kv_fp8) launch_dma<EPI_QKV8, 2, 4>(s, A, Wp, nullptr, M, N, K, 1, nullptr, nullptr, 0.f, q);
    else launch_dma<EPI_QKV, 2, 4>(s, A, Wp, nullptr, M, N, K, 1, nullptr, nullptr, 0.f, q);
  } else {
    if (kv_fp8) launch_dma<EPI_QKV8, 4, 4>(s, A, Wp, nullptr, M, N, K, 1, nullptr, nullptr, 0.f, q);
    else launch_dma<EPI_QKV, 4, 4>(s, A, Wp, nullptr, M, N, K, 1, nullptr, nullptr, 0.f, q);
  }
}

// lm-head of a decode step: logits[M, V] (fp32, row-major) and, unless null, stripmax[M, V / 32]; the logits are the same
// bits either way.
void launch_lm_head_logits(hipStream_t s, const bf16_t* A, const bf16_t* Wp, float* logits, int M,
                           int V, int K, float* stripmax) {
  if (M <= 0) return;
  if (stripmax) gemm_launch<EPI_STORE_MAX>(s, A, Wp, logits, M, V, K, 1, K / 64, stripmax, 0.f);
  else gemm_launch<EPI_STORE>(s, A, Wp, logits, M, V, K, 1, K / 64, nullptr, 0.f);
}

// One workgroup per row: combine the per-strip (max, sum) pairs in a fixed order and write
// log softmax(z / T)[target] = (z_t - max) c ln2 - ln sum, c = log2(e) / T.
__global__ __launch_bounds__(256) void lse_finish_kernel(const float2* __restrict__ P,
                                                         const float* __restrict__ zt, int NB,
                                                         float scale_c, float* __restrict__ lp) {
  __shared__ float red[4];
  const int row = blockIdx.x, tid = threadIdx.x;
  const float2* p = P + (size_t)row * NB;
  float mx = -3.0e38f;
  for (int j = tid; j < NB; j += 256) mx = fmaxf(mx, p[j].x);
  mx = wave_max(mx);
  if ((tid & 63) == 0) red[tid >> 6] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  __syncthreads();
  float sm = 0.f;
  for (int j = tid; j < NB; j += 256) {
    float2 v = p[j];
    sm += v.y * exp2f((v.x - mx) * scale_c);
  }
  sm = wave_sum(sm);
  if ((tid & 63) == 0) red[tid >> 6] = sm;
  __syncthreads();
  if (tid == 0) {
    float S = (red[0] + red[1]) + (red[2] + red[3]);
    lp[row] = (zt[row] - mx) * scale_c * 0.6931471805599453f - logf(S);
  }
}

void launch_lm_head_logprob(hipStream_t s, const bf16_t* A, const bf16_t* Wp, int M, int V, int K,
                            const int32_t* tgt, float scale_c, float* part, float* zt, float* lp) {
  if (M <= 0) return;
  if (plan_gemm(M, V, K, EPI_LSE, 0).kind == GEMM_TILE256) {
    launch_dma<EPI_LSE, 4, 4>(s, A, Wp, part, M, V, K, 1, tgt, zt, scale_c, QkvArgs{});
  } else {
    dim3 grid((V + 127) / 128, (M + 127) / 128, 1);
    gemm_mfma_kernel<EPI_LSE, 4, false><<<grid, 256, 0, s>>>(A, Wp, part, M, V, K, K / 64, tgt, zt, scale_c);
  }
  lse_finish_kernel<<<M, 256, 0, s>>>((const float2*)part, zt, V / 32, scale_c, lp);
}

// =============================================================================================
// Paged GQA attention, one workgroup (4 waves) per (work item, kv head, context split).
// The MFMA column index n = G * r + hq carries query row r of the item and query head hq of the kv
// head's group of G = n_q / n_kv heads (G a power of two <= 16, r < 16 / G), so decode (1 row) and
// chunked prefill (16 / G rows) share the kernel.
// Per 16-token page:  S^T[token, n] = K[token, :] . Q[n, :]   (4 x mfma 16x16x32, K straight from
// the page in operand order), online softmax per column, O^T[d, n] += V^T[d, token] P^T[token, n]
// (8 x mfma 16x16x16; the score accumulator layout is exactly the P operand layout).
// The item's page range is split over the 4 waves; partial (max, sum, O) are merged in fixed order
// through LDS and, when a row's context was cut into several items, through a scratch buffer and a
// second kernel.
// =============================================================================================
#define ATT_NEG (-1.0e30f)

// One page of the online-softmax loop; see the kernels below for the variables they use.
// Two flavours of the page load.  The decode kernel reads a trajectory's own pages once per step:
// those loads carry the non-temporal hint (measured 8-10 % more bandwidth than plain loads).  Pages
// shared with other trajectories of the step (a forked prompt) keep plain loads so that the group
// finds them in L2, and so does the prefill kernel, which re-reads pages across waves and items.
// The choice is made per wave, outside the page loop: inside it the compiler would merge the two
// loads into one and drop the hint.
// kpool / vpool are byte pointers; a (page, kv head) block is BLK bytes (4096: bf16, 2048: 8-bit
// cache) that a wave reads as NLD 16-byte slots per lane (head_off = kv head * BLK + lane * 16).
#define ATT_LOAD_PLAIN(KR, VR, IDX, ORDER)                                     \
  {                                                                           \
    const size_t base_ = (size_t)((uint64_t)(uint32_t)__builtin_amdgcn_readlane(ids, IDX) * (uint32_t)(nkv * BLK)); \
    _Pragma("unroll") for (int c = 0; c < NLD; c++) {                         \
      KR[c] = *(const u32x4*)(khead + base_ + (lane16 + c * 1024));           \
      VR[c] = *(const u32x4*)(vhead + base_ + (lane16 + c * 1024));           \
      ORDER                                                                   \
    }                                                                         \
  }
#define ATT_LOAD_STREAM(KR, VR, IDX, ORDER)                                    \
  {                                                                           \
    const size_t base_ = (size_t)((uint64_t)(uint32_t)__builtin_amdgcn_readlane(ids, IDX) * (uint32_t)(nkv * BLK)); \
    _Pragma("unroll") for (int c = 0; c < NLD; c++) {                         \
      KR[c] = __builtin_nontemporal_load((const u32x4*)(khead + base_ + (lane16 + c * 1024))); \
      VR[c] = __builtin_nontemporal_load((const u32x4*)(vhead + base_ + (lane16 + c * 1024))); \
      ORDER                                                                   \
    }                                                                         \
  }
// Operand register i of a page buffer: the 16-byte slot itself (bf16 cache), or half a raw slot
// of the 8-bit cache widened to bf16 (exact) just before use, so that no widened page stays live.
template <bool FP8, int N>
__device__ __forceinline__ u32x4 att_operand(const u32x4 (&R)[N], int i) {
  if constexpr (FP8) {
    uint32_t a, b, c, d;
    e4m3x4_to_bf16(R[i >> 1][2 * (i & 1)], &a, &b);
    e4m3x4_to_bf16(R[i >> 1][2 * (i & 1) + 1], &c, &d);
    return (u32x4){a, b, c, d};
  } else {
    return R[i];
  }
}
#define ATT_PAGE(KR, VR, PG)                                                  \
  {                                                                           \
    f32x4 S = (f32x4){0.f, 0.f, 0.f, 0.f};                                    \
    _Pragma("unroll") for (int c = 0; c < 4; c++)                             \
      S = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, att_operand<FP8>(KR, c)), \
                                                  __builtin_bit_cast(bf16x8, qreg[c]), S, 0, 0, 0); \
    float sv[4], mx = ATT_NEG;                                                \
    bool vis[4];                                                              \
    _Pragma("unroll") for (int i = 0; i < 4; i++) {                           \
      int tg = (PG) * RL_PAGE + 4 * g + i;                                    \
      vis[i] = colvalid && tg <= mypos && (PG) < pg1;                         \
      sv[i] = vis[i] ? S[i] * scale2 : ATT_NEG;                               \
      mx = fmaxf(mx, sv[i]);                                                  \
    }                                                                         \
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));                                   \
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));                                   \
    float mn = fmaxf(m, mx);                                                  \
    float alpha = exp2f(m - mn);                                              \
    float ps = 0.f;                                                           \
    s16x4 pb;                                                                 \
    _Pragma("unroll") for (int i = 0; i < 4; i++) {                           \
      float p = vis[i] ? exp2f(sv[i] - mn) : 0.f;                             \
      ps += p;                                                                \
      pb[i] = (short)f2bf(p);                                                 \
    }                                                                         \
    l = l * alpha + ps;                                                       \
    m = mn;                                                                   \
    _Pragma("unroll") for (int jp = 0; jp < 4; jp++) {                        \
      s16x4 v0, v1;                                                           \
      const u32x4 vr_ = att_operand<FP8>(VR, jp);                             \
      v0[0] = (short)(vr_[0] & 0xffff); v0[1] = (short)(vr_[0] >> 16);        \
      v0[2] = (short)(vr_[1] & 0xffff); v0[3] = (short)(vr_[1] >> 16);        \
      v1[0] = (short)(vr_[2] & 0xffff); v1[1] = (short)(vr_[2] >> 16);        \
      v1[2] = (short)(vr_[3] & 0xffff); v1[3] = (short)(vr_[3] >> 16);        \
      _Pragma("unroll") for (int i = 0; i < 4; i++) { acc[2 * jp][i] *= alpha; acc[2 * jp + 1][i] *= alpha; } \
      acc[2 * jp] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(v0, pb, acc[2 * jp], 0, 0, 0); \
      acc[2 * jp + 1] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(v1, pb, acc[2 * jp + 1], 0, 0, 0); \
    }                                                                         \
  }
// Order of a page step of the decode kernel: (2 loads, 1 MFMA) x 4, everything else after.
#define ATT_SPREAD                                                            \
  __builtin_amdgcn_sched_group_barrier(0x020, 2, 0);                          \
  __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                          \
  __builtin_amdgcn_sched_group_barrier(0x020, 2, 0);                          \
  __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                          \
  __builtin_amdgcn_sched_group_barrier(0x020, 2, 0);                          \
  __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                          \
  __builtin_amdgcn_sched_group_barrier(0x020, 2, 0);                          \
  __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
// The decode kernel's page loop (uses pt, pg0, pg1, pglast, lane, lane16, khead, vhead, nkv and the
// buffers kA, vA, kB, vB of the enclosing kernel); LOAD is one of the two load macros.
// The wave's page-table entries lie in one register, entry i of 64 in lane i (ATT_IDS).  Requested page by page, an entry's sign
// extension stood right behind its load, and every second page waited for all that was in flight.  A decode step of 8 layers: 16 rows
// over 1000 keys (16 heads over 8) 430 -> 403 us, 4 over 3000 402 -> 392, 8-bit cache (32 heads over 8) 32 over 3000 891 -> 867; from 32
// rows over 3000 keys of the bf16 cache on, where the memory is busy all the time, within 1 %.
// Loads in the order written, ahead of the loop as in it: where the compiler had turned the first page's around, the wait for a page's
// first key block, the longer one of both ways into the loop, was a wait for its last value block.
#define ATT_ORDER __builtin_amdgcn_sched_barrier(0);
#define ATT_IDS(PG)                                                           \
  {                                                                           \
    pgb = (PG);                                                               \
    ids = pt[min(pgb + lane, pglast)];                                        \
    asm volatile("" : "+v"(ids));   /* arrives here, not at every use */      \
  }
#define ATT_PAGE_LOOP(LOAD)                                                   \
  if (pg0 < pg1) {                                                            \
    int pgb, ids;                                                             \
    ATT_IDS(pg0)                                                              \
    LOAD(kA, vA, 0, ATT_ORDER)                                                           \
    for (int pg = pg0; pg < pg1; pg += 2) {                                   \
      if (pg - pgb > 64 - 3) ATT_IDS(pg)                                      \
      __builtin_amdgcn_sched_barrier(0);                                      \
      /* page pg is in A; pg+1 -> B.  The eight loads of a page are issued two at a time between the four score MFMAs of the \
         page being consumed (ATT_SPREAD) rather than in one burst: +0.5-2 % bandwidth. */ \
      LOAD(kB, vB, pg + 1 - pgb, )                                              \
      ATT_PAGE(kA, vA, pg)                                                \
      ATT_SPREAD                                                              \
      __builtin_amdgcn_sched_barrier(0);                                      \
      /* page pg+1 is in B; pg+2 -> A */                                      \
      LOAD(kA, vA, pg + 2 - pgb, )                                              \
      ATT_PAGE(kB, vB, pg + 1)                                            \
      ATT_SPREAD                                                              \
      __builtin_amdgcn_sched_barrier(0);                                      \
    }                                                                         \
  }

// The same loop three pages deep (buffers A-C; two pages in flight while one is consumed), used
// with the 8-bit cache: its pages are half as large, and one of them in flight per wave no longer
// covers the memory latency.
#define ATT_PAGE_LOOP3(LOAD)                                                  \
  if (pg0 < pg1) {                                                            \
    int pgb, ids;                                                             \
    ATT_IDS(pg0)                                                              \
    LOAD(kA, vA, 0, ATT_ORDER)                                                           \
    LOAD(kB, vB, 1, ATT_ORDER)                                                           \
    for (int pg = pg0; pg < pg1; pg += 3) {                                   \
      if (pg - pgb > 64 - 5) ATT_IDS(pg)                                      \
      LOAD(kC, vC, pg + 2 - pgb, ATT_ORDER)                                              \
      __builtin_amdgcn_sched_barrier(0);                                      \
      ATT_PAGE(kA, vA, pg)                                                \
      __builtin_amdgcn_sched_barrier(0);                                      \
      LOAD(kA, vA, pg + 3 - pgb, ATT_ORDER)                                              \
      __builtin_amdgcn_sched_barrier(0);                                      \
      ATT_PAGE(kB, vB, pg + 1)                                            \
      __builtin_amdgcn_sched_barrier(0);                                      \
      LOAD(kB, vB, pg + 4 - pgb, ATT_ORDER)                                              \
      __builtin_amdgcn_sched_barrier(0);                                      \
      ATT_PAGE(kC, vC, pg + 2)                                            \
      __builtin_amdgcn_sched_barrier(0);                                      \
    }                                                                         \
  }

// row_stride: floats between the outputs of two MFMA columns of one part
__device__ __forceinline__ void attn_merge_store(const float* __restrict__ pm,
                                                 const float* __restrict__ pl,
                                                 const float* __restrict__ pacc, int nparts,
                                                 size_t part_stride_ml, size_t part_stride_acc,
                                                 int row_stride, int n, int d0, float* m_out,
                                                 float* l_out, float* o8) {
  float mt = ATT_NEG;
  for (int w = 0; w < nparts; w++) mt = fmaxf(mt, pm[w * part_stride_ml + n]);
  float L = 0.f;
#pragma unroll
  for (int e = 0; e < 8; e++) o8[e] = 0.f;
  for (int w = 0; w < nparts; w++) {
    float f = exp2f(pm[w * part_stride_ml + n] - mt);
    L += f * pl[w * part_stride_ml + n];
    const float* a = pacc + w * part_stride_acc + (size_t)n * row_stride + d0;
#pragma unroll
    for (int e = 0; e < 8; e++) o8[e] += f * a[e];
  }
  *m_out = mt;
  *l_out = L;
}

// ROPE (single-row items, one row of a trajectory): 0, or the kernel starts from the projection's partial sums (2: rows not yet divided
// by their rms): sixteen lanes per head form the group's queries, and in the workgroup that reads the row's last page also its key and
// value, which go to that page before that workgroup, the only one to use them, reads it.  Every part of a row forms the same
// queries.  See attention_takes_rope.
template <bool FP8, int ROPE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void attention_mfma_kernel(
    const bf16_t* __restrict__ q, char* kpool, char* vpool,
    const AttnItem* __restrict__ items, const int32_t* __restrict__ rowlist,
    const int32_t* __restrict__ page_table, bf16_t* __restrict__ o, float* __restrict__ scratch,
    int nq, int nkv, int gshift, int pt_stride, float scale2, RopeArgs rope) {
  // a column's 128 outputs are padded to 132 floats: with a stride of 128 the 16 lanes that hold
  // one token group's 16 columns would all store into the same 4 banks
  constexpr int AST = 132;
  __shared__ __align__(16) float s_acc[4 * 16 * AST];
  __shared__ float s_m[4 * 16];
  __shared__ float s_l[4 * 16];
  // blockIdx.x = item * nkv + kvh: consecutive workgroups go round-robin to the 8 XCDs, so with
  // kv head fastest all trajectories of one kv head share an XCD (for nkv = 8) and trajectories
  // that share prompt pages (a forked group, adjacent items) find each other's pages in that L2.
  const int item_idx = blockIdx.x / nkv;
  const AttnItem it = items[item_idx];
  const int kvh = blockIdx.x - item_idx * nkv;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int g = lane >> 4, n = lane & 15, r = n >> gshift, hq = n & ((1 << gshift) - 1);
  const bool colvalid = r < it.nrows;
  // shared-prefix items: every page of the range lies before every member's position
  const bool gather = (it.gather & 1) != 0;
  const int mypos = gather ? 0x3fffffff : it.pos0 + r;
  const int qrow = !colvalid ? 0 : (gather ? rowlist[it.row0 + r] : it.row0 + r);
  const int per = (it.pg_hi - it.pg_lo + 3) >> 2;
  const int pg0 = it.pg_lo + wave * per, pg1 = min(pg0 + per, it.pg_hi);
  const int32_t* pt = page_table + (size_t)it.slot * pt_stride;

  u32x4 qreg[4];
  if constexpr (ROPE != 0) {
    __shared__ __align__(16) bf16_t s_q[8][128];
    const int grp = tid >> 4, sub = tid & 15, G = 1 << gshift, last = it.pos0 / RL_PAGE;
    const int hd = grp < G ? (kvh << gshift) + grp : nq + (grp - G) * nkv + kvh;      // the group's queries, then its key and its value
    if (grp < G || (grp < G + 2 && it.pg_hi > last)) {
      uint2 w1, w2;
      qkrope_head128<FP8, ROPE == 2>(rope, it.row0, hd, sub, it.pos0, [&] { return pt[last]; }, (bf16_t*)kpool, (bf16_t*)vpool, &w1, &w2);
      if (grp < G) {
        *(uint2*)&s_q[grp][sub * 4] = w1;
        *(uint2*)&s_q[grp][64 + sub * 4] = w2;
      }
    }
    __syncthreads();      // the key and the value are stored, too
#pragma unroll
    for (int c = 0; c < 4; c++) {
      qreg[c] = (u32x4){0u, 0u, 0u, 0u};
      if (colvalid) qreg[c] = *(const u32x4*)&s_q[hq][c * 32 + g * 8];
    }
  } else {
#pragma unroll
    for (int c = 0; c < 4; c++) {
      qreg[c] = (u32x4){0u, 0u, 0u, 0u};
      if (colvalid)
        qreg[c] = *(const u32x4*)(q + ((size_t)qrow * nq + ((kvh << gshift) + hq)) * 128 + c * 32 + g * 8);
    }
  }
  f32x4 acc[8];
#pragma unroll
  for (int j = 0; j < 8; j++) acc[j] = (f32x4){0.f, 0.f, 0.f, 0.f};
  float m = ATT_NEG, l = 0.f;

  // Two page buffers (A, B) alternate: while one page is consumed the next one is already on its
  // way, and the page-table entry after that has been requested.  Loads past the end of this
  // wave's range are clamped to its last page (a re-read that hits in cache) so that nothing in
  // the loop defines registers conditionally; sched_barrier keeps the loads where they are
  // written, ahead of the arithmetic.
  const int pglast = max(pg1 - 1, pg0);
  constexpr int NLD = FP8 ? 2 : 4, BLK = FP8 ? 2048 : 4096;
  const char *const khead = kpool + (size_t)kvh * BLK, *const vhead = vpool + (size_t)kvh * BLK;
  const uint32_t lane16 = lane * 16;
  u32x4 kA[NLD], vA[NLD], kB[NLD], vB[NLD];
  // a wave whose share of the pages starts behind the trajectory's shared leading pages streams
  if constexpr (FP8) {
    u32x4 kC[NLD], vC[NLD];
    if (pg0 >= (it.gather >> 8)) {
      ATT_PAGE_LOOP3(ATT_LOAD_STREAM)
    } else {
      ATT_PAGE_LOOP3(ATT_LOAD_PLAIN)
    }
  } else {
    if (pg0 >= (it.gather >> 8)) {
      ATT_PAGE_LOOP(ATT_LOAD_STREAM)
    } else {
      ATT_PAGE_LOOP(ATT_LOAD_PLAIN)
    }
  }
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  // wave partials -> LDS: acc[jb][i] is O^T[d = 16 jb + 4 g + i][column n]
#pragma unroll
  for (int jb = 0; jb < 8; jb++) *(f32x4*)&s_acc[(wave * 16 + n) * AST + jb * 16 + g * 4] = acc[jb];
  if (g == 0) { s_m[wave * 16 + n] = m; s_l[wave * 16 + n] = l; }
  __syncthreads();
  // 256 threads: column cn = tid / 16, dims d0 .. d0+7
  const int cn = tid >> 4, d0 = (tid & 15) * 8;
  float mt, L, o8[8];
  attn_merge_store(s_m, s_l, s_acc, 4, 16, 16 * AST, AST, cn, d0, &mt, &L, o8);
  const int cr = cn >> gshift, chq = cn & ((1 << gshift) - 1);
  if (it.part < 0) {
    if (cr < it.nrows) {
      float inv = 1.0f / L;
      uint32_t w[4];
#pragma unroll
      for (int e = 0; e < 4; e++)
        w[e] = (uint32_t)f2bf(o8[2 * e] * inv) | ((uint32_t)f2bf(o8[2 * e + 1] * inv) << 16);
      *(uint4*)(o + atile_off(it.row0 + cr, ((kvh << gshift) + chq) * 128 + d0, nq * 128)) =
          make_uint4(w[0], w[1], w[2], w[3]);
    }
  } else {
    float* dst = scratch + ((size_t)it.part * nkv + kvh) * (16 * 130);
#pragma unroll
    for (int e = 0; e < 8; e++) dst[cn * 128 + d0 + e] = o8[e];
    if ((tid & 15) == 0) { dst[16 * 128 + cn] = mt; dst[16 * 128 + 16 + cn] = L; }
  }
}

// Chunked prefill: one workgroup per (item of up to 4 * 32/G rows, kv head), a wave = 32 columns
// (query row, head of the group), 32x32x16 MFMAs.  A pair of pages (32 keys) is a stage of 16 KB in LDS (8-bit cache: 8 KB), loaded
// there directly in the pool's operand order (no registers, no LDS stores), two pairs ahead in a ring of three:
//   S^T[32 keys, 32 columns] = K . Q^T, 8 steps of 16 dims: lane (key, half) reads its 8 dims of a step as 16 bytes (8-bit cache:
//   of two steps), 16 keys of a page being 256 contiguous bytes;
//   O^T[32 dims, 32 columns] += V^T . P^T in two steps of 16 keys, per block of 32 dims: lane l of the scores holds, for column
//   l % 32, keys 8 j + 4 (l / 32) + 0 .. 3 (j = 0, 1: first page, 2, 3: second).  Step x takes j = x and j = 2 + x, so a lane's eight
//   slots are four keys of either page on both sides, and the values are two 8-byte reads a page apart, 64 lanes covering 512
//   contiguous bytes.  Key group 2 x + l / 32, these eight keys, has its own fp32 sum of the terms before they are rounded.
// Nothing is moved between registers to put an operand together.  One barrier per pair: behind it the pair is complete for
// every wave and the stage of the pair before is free for the pair after the next.
// What bounds it: a wave's matrix and vector work take turns (32 keys x 32 columns: 512 cycles of MFMA, 61 vector instructions
// of which 16 exponentials), so other waves of the SIMD have to fill the pipes, and three fit the registers (155; 8-bit cache 150); then
// power.  Over 3300 keys the matrix pipes are busy 0.48 of the time, LDS 0.60 of which 0.24 are bank conflicts, at 1.9 GHz; on operands of
// zeros 12 x 610 rows over 3000 keys take 330 us, on random ones 421 (0.94 PFLOP/s).  Before, with 16x16x32 MFMAs, two waves a SIMD, keys
// and values through registers and the pages' addresses formed by every lane: 418 and 502; 16 x 512 rows over none 87 -> 78 us,
// 24 x 340 over 2000 with two heads a group 227 -> 179, 8-bit cache 515 -> 432 (all from traces of engine passes).
// Items are taken from the last to the first: a trajectory's later rows see more keys, and short items fill the end of the launch
// better (8 x 1024 rows over none 105 -> 99 us).
// Page indices past the item's last page are clamped to it (their keys are masked: they lie
// behind every row of the item); the pool is cleared at load, so such blocks hold finite values.
template <bool FP8, bool MASKED>
__device__ __forceinline__ void prefill_pair(const char* kb, const char* vb, int key0, const u32x4 (&q)[8], f32x16 (&acc)[4],
                                             float& m, float (&l)[2], int mypos, float scale2, int lane) {
  f32x16 S;
#pragma unroll
  for (int i = 0; i < 16; i++) S[i] = 0.f;
  auto score = [&](const u32x4& k, int ks) {
    S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, k), __builtin_bit_cast(bf16x8, q[ks]), S, 0, 0, 0);
  };
  if constexpr (FP8) {
#pragma unroll
    for (int x = 0; x < 2; x++) {      // a slot holds the lane's dims of steps ks and ks + 2; steps in ascending order
      const u32x4 raw[2] = {*(const u32x4*)(kb + x * 1024), *(const u32x4*)(kb + x * 1024 + 512)};
#pragma unroll
      for (int ks = 0; ks < 4; ks++) {
        const u32x4 one[1] = {raw[ks & 1]};
        score(att_operand<true>(one, ks >> 1), 4 * x + ks);
      }
    }
  } else {
#pragma unroll
    for (int ks = 0; ks < 8; ks++) score(*(const u32x4*)(kb + ks * 512), ks);
  }
  // m (in scaled units: score * scale2, scale2 > 0) is the reference point of the exponents, not
  // necessarily the running maximum: it only moves, to the column's maximum so far, when the eight terms of a key group
  // in some column of the 16 around it sum to more than kLazy = 2^8.  The ratio acc / l does not depend on m, and the common
  // case needs neither a maximum nor a rescaling: the terms are formed first, and their sums, which
  // are needed anyway, show whether one of them was that large (or infinite: they are formed again).
  constexpr float kLazy = 256.0f;
  typedef __attribute__((__vector_size__(4))) __bf16 bf16x2;
  union { bf16x2 pair[8]; bf16x8 P[2]; } t;
  float ps[2];
  auto vis = [&](int i) { return !MASKED || key0 + (i >> 2) * 8 + (i & 3) <= mypos; };
  auto terms = [&]() {
#pragma unroll
    for (int x = 0; x < 2; x++) {
      float p[8];
#pragma unroll
      for (int e = 0; e < 8; e++) {
        const int i = (e >> 2) * 8 + 4 * x + (e & 3);
        p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(S[i], scale2, -m));
        if (MASKED) p[e] = vis(i) ? p[e] : 0.f;
      }
      ps[x] = ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
#pragma unroll
      for (int e = 0; e < 4; e++) t.pair[4 * x + e] = (bf16x2){(__bf16)p[2 * e], (__bf16)p[2 * e + 1]};
    }
  };
  terms();
  if (const uint64_t hit = __ballot(ps[0] > kLazy || ps[1] > kLazy)) {
    const bool moves = hit & ((lane & 16) ? 0xffff0000ffff0000ull : 0x0000ffff0000ffffull);
    float mx = ATT_NEG;
#pragma unroll
    for (int i = 0; i < 16; i++) mx = fmaxf(mx, vis(i) ? S[i] : ATT_NEG);
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mn = moves ? fmaxf(m, mx * scale2) : m;
    const float alpha = exp2f(m - mn);
    l[0] *= alpha;
    l[1] *= alpha;
#pragma unroll
    for (int j = 0; j < 4; j++)
#pragma unroll
      for (int i = 0; i < 16; i++) acc[j][i] *= alpha;
    m = mn;
    terms();
  }
  l[0] += ps[0];
  l[1] += ps[1];
  auto value = [&](int x, int db) {
    if constexpr (FP8) {
      const char* at = vb + x * 512 + (db >> 1) * 1024 + (db & 1) * 8;
      uint32_t a, b, c, d;
      e4m3x4_to_bf16(*(const uint32_t*)at, &a, &b);
      e4m3x4_to_bf16(*(const uint32_t*)(at + 2048), &c, &d);
      return (u32x4){a, b, c, d};
    } else {
      const char* at = vb + x * 512 + db * 1024;
      const uint2 lo = *(const uint2*)at, hi = *(const uint2*)(at + 4096);
      asm volatile("" ::: "memory");      // joined with another read's, the halves would have to be moved (24 moves)
      return (u32x4){lo.x, lo.y, hi.x, hi.y};
    }
  };
  auto add = [&](const u32x4& v, int x, int db) {
    acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, v), t.P[x], acc[db], 0, 0, 0);
  };
  u32x4 v[2][4];
#pragma unroll
  for (int db = 0; db < 4; db++) v[0][db] = value(0, db);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int db = 0; db < 4; db++) {
    v[1][db] = value(1, db);
    add(v[0][db], 0, db);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int db = 0; db < 4; db++) add(v[1][db], 1, db);
}

template <bool FP8>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void attention_prefill_kernel(
    const bf16_t* __restrict__ q, const char* __restrict__ kpool, const char* __restrict__ vpool,
    const AttnItem* __restrict__ items, const int32_t* __restrict__ page_table,
    bf16_t* __restrict__ o, int nq, int nkv, int gshift, int pt_stride, float scale2) {
  constexpr int BLK = FP8 ? 2048 : 4096, R = 3, STAGE = 4 * BLK;         // key blocks of the two pages, then value blocks
  constexpr int NL = BLK / 1024;                                         // loads of a wave and stage
  __shared__ __align__(16) char s_kv[R * STAGE];
  const int back = blockIdx.x / nkv, kvh = blockIdx.x - back * nkv;
  const AttnItem it = items[gridDim.x / nkv - 1 - back];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int n = lane & 31, half = lane >> 5, head = (kvh << gshift) + (n & ((1 << gshift) - 1));
  const int rpw = 32 >> gshift;                       // rows of a wave
  const int wrow0 = wave * rpw, wave_rows = min(it.nrows - wrow0, rpw);
  const int pg1 = wave_rows > 0 ? (it.pos0 + wrow0 + wave_rows - 1) / RL_PAGE + 1 : 0;
  const int pglast = (it.pos0 + it.nrows - 1) / RL_PAGE;
  const int nst = (pglast + 2) / 2;
  // pages that end at or before the wave's first row are visible to all of its rows: no masking
  const int full_pages = wave_rows > 0 ? (it.pos0 + wrow0 + 1) / RL_PAGE : 0;
  const int32_t* pt = page_table + (size_t)it.slot * pt_stride;
  const int r = wrow0 + (n >> gshift);
  // columns past the item's rows get position -1: every key of a masked pair is masked for them
  const int mypos = r < it.nrows ? it.pos0 + r : -1;
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void*)s_kv;
  // (a pool holds less than 2^32 (page, kv head) blocks)
  auto block = [&](int pg) { return (size_t)((unsigned)pt[min(pg, pglast)] * (unsigned)nkv + (unsigned)kvh) * BLK; };
  // this wave's share of a stage: a quarter of each of its four blocks, or with the 8-bit cache half of one page's two
  auto load = [&](int buf, size_t b0, size_t b1) {
    const unsigned dst = lds0 + (unsigned)buf * STAGE, part = (unsigned)(FP8 ? wave & 1 : wave) * 1024u;
    if constexpr (FP8) {
      const size_t b = wave < 2 ? b0 : b1;
      const unsigned at = dst + (wave < 2 ? 0u : 2048u) + part;
      load_to_lds(at, lane * 16, buffer_rsrc(kpool + b, BLK), part);
      load_to_lds(at + 4096u, lane * 16, buffer_rsrc(vpool + b, BLK), part);
    } else {
      load_to_lds(dst + part, lane * 16, buffer_rsrc(kpool + b0, BLK), part);
      load_to_lds(dst + 4096u + part, lane * 16, buffer_rsrc(kpool + b1, BLK), part);
      load_to_lds(dst + 8192u + part, lane * 16, buffer_rsrc(vpool + b0, BLK), part);
      load_to_lds(dst + 12288u + part, lane * 16, buffer_rsrc(vpool + b1, BLK), part);
    }
  };
  u32x4 qr[8];
#pragma unroll
  for (int ks = 0; ks < 8; ks++) {
    qr[ks] = (u32x4){0u, 0u, 0u, 0u};
    if (r < it.nrows) qr[ks] = *(const u32x4*)(q + ((size_t)(it.row0 + r) * nq + head) * 128 + ks * 16 + half * 8);
  }
#pragma unroll
  for (int ks = 0; ks < 8; ks++) asm volatile("" : "+v"(qr[ks]));      // they have arrived before the loads that the loop counts
  f32x16 acc[4];
#pragma unroll
  for (int j = 0; j < 4; j++)
#pragma unroll
    for (int i = 0; i < 16; i++) acc[j][i] = 0.f;
  float m = ATT_NEG, l[2] = {0.f, 0.f};
  load(0, block(0), block(1));
  load(1, block(2), block(3));
  size_t n0 = block(4), n1 = block(5);
  const char* kl = s_kv + (n >> 4) * BLK + (n & 15) * 16 + half * 256;
  const char* vl = s_kv + 2 * BLK + (n & 15) * 16 + (n >> 4) * (FP8 ? 4 : 8) + half * 256;
  int buf = 0;
  // pair s is there for every wave, and pair s - 1 is read out by every wave: pair s + 2 takes its stage
  auto advance = [&](int s) {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(NL) : "memory");
    __builtin_amdgcn_s_barrier();
    load(buf == 0 ? 2 : buf - 1, n0, n1);
    n0 = block(2 * s + 6);
    n1 = block(2 * s + 7);
  };
  // (two loops: with the choice inside one the accumulators are copied between the two forms)
  const int nfull = full_pages >> 1;
  for (int s = 0; s < nfull; s++) {
    advance(s);
    prefill_pair<FP8, false>(kl + buf * STAGE, vl + buf * STAGE, 0, qr, acc, m, l, mypos, scale2, lane);
    buf = buf == 2 ? 0 : buf + 1;
  }
  for (int s = nfull; s < nst; s++) {
    advance(s);
    if (2 * s < pg1)
      prefill_pair<FP8, true>(kl + buf * STAGE, vl + buf * STAGE, 2 * s * RL_PAGE + 4 * half, qr, acc, m, l, mypos, scale2, lane);
    buf = buf == 2 ? 0 : buf + 1;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  const float sum = (l[0] + __shfl_xor(l[0], 32, 64)) + (l[1] + __shfl_xor(l[1], 32, 64));
  if (r >= it.nrows) return;
  // acc[db][i] is O[row r][head][d = 32 db + (i / 4) * 8 + 4 half + i % 4]: four consecutive dims = one 8-byte store
  const float inv = 1.0f / sum;
#pragma unroll
  for (int db = 0; db < 4; db++)
#pragma unroll
    for (int j = 0; j < 4; j++) {
      uint2 w;
      w.x = (uint32_t)f2bf(acc[db][4 * j] * inv) | ((uint32_t)f2bf(acc[db][4 * j + 1] * inv) << 16);
      w.y = (uint32_t)f2bf(acc[db][4 * j + 2] * inv) | ((uint32_t)f2bf(acc[db][4 * j + 3] * inv) << 16);
      *(uint2*)(o + atile_off(it.row0 + r, head * 128 + 32 * db + 8 * j + 4 * half, nq * 128)) = w;
    }
}

// grid (n_merges, nkv), block 256: merge the parts of one (row, kv head): the shared-prefix parts (the
// row is row `sr` of those items), then the row's own parts.  16 lanes hold a head's 128 outputs; the
// 16 such lane groups are dealt over the G heads and over 16/G shares of the parts (share x takes parts
// x, x + 16/G, ...), four parts' reads in flight at a time, and the shares are added through LDS in
// ascending order: a chain of a few reads instead of two per part (6 rows x 8 kv heads of ~24 parts:
// 16.1 -> 3.8 us).
__global__ __launch_bounds__(256) void attention_merge_kernel(const float* __restrict__ scratch,
                                                              const AttnMerge* __restrict__ merges,
                                                              bf16_t* __restrict__ o, int nq,
                                                              int nkv, int gshift) {
  __shared__ __align__(16) float s_o[16][132];
  __shared__ float s_m[16], s_l[16];
  const AttnMerge mg = merges[blockIdx.x];
  const int kvh = blockIdx.y, tid = threadIdx.x;
  const int grp = tid >> 4, d0 = (tid & 15) * 8;
  const int hq = grp & ((1 << gshift) - 1), share = grp >> gshift, nshare = 16 >> gshift;
  const int total = mg.snparts + mg.nparts;
  const int scol = (mg.sr << gshift) + hq;
  // part w: slot and column holding this row's head hq
  auto src_of = [&](int w, int* col) -> const float* {
    const bool sh = w < mg.snparts;
    *col = sh ? scol : hq;
    const int slot = sh ? mg.sfirst + w : mg.first + (w - mg.snparts);
    return scratch + ((size_t)slot * nkv + kvh) * (16 * 130);
  };
  float mt = ATT_NEG, L = 0.f, o8[8];
#pragma unroll
  for (int e = 0; e < 8; e++) o8[e] = 0.f;
  for (int w0 = share; w0 < total; w0 += 4 * nshare) {
    float pm[4], pl[4];
    f32x4 a0[4], a1[4];
#pragma unroll
    for (int j = 0; j < 4; j++) {
      const int w = w0 + j * nshare;
      int col;
      const float* src = src_of(min(w, total - 1), &col);
      pm[j] = src[16 * 128 + col];
      pl[j] = src[16 * 128 + 16 + col];
      a0[j] = *(const f32x4*)(src + (size_t)col * 128 + d0);
      a1[j] = *(const f32x4*)(src + (size_t)col * 128 + d0 + 4);
    }
    float mn = mt;
#pragma unroll
    for (int j = 0; j < 4; j++) {
      if (w0 + j * nshare < total) mn = fmaxf(mn, pm[j]);
    }
    const float f = exp2f(mt - mn);
    L *= f;
#pragma unroll
    for (int e = 0; e < 8; e++) o8[e] *= f;
#pragma unroll
    for (int j = 0; j < 4; j++) {
      if (w0 + j * nshare >= total) continue;
      const float fj = exp2f(pm[j] - mn);
      L += fj * pl[j];
#pragma unroll
      for (int e = 0; e < 4; e++) { o8[e] += fj * a0[j][e]; o8[4 + e] += fj * a1[j][e]; }
    }
    mt = mn;
  }
  *(f32x4*)&s_o[grp][d0] = (f32x4){o8[0], o8[1], o8[2], o8[3]};
  *(f32x4*)&s_o[grp][d0 + 4] = (f32x4){o8[4], o8[5], o8[6], o8[7]};
  if ((tid & 15) == 0) { s_m[grp] = mt; s_l[grp] = L; }
  __syncthreads();
  if (share != 0) return;
  float M = mt;
  for (int x = 1; x < nshare; x++) M = fmaxf(M, s_m[(x << gshift) + hq]);
  float f = exp2f(mt - M);
  L *= f;
#pragma unroll
  for (int e = 0; e < 8; e++) o8[e] *= f;
  for (int x = 1; x < nshare; x++) {
    const int gx = (x << gshift) + hq;
    f = exp2f(s_m[gx] - M);
    L += f * s_l[gx];
    const f32x4 b0 = *(const f32x4*)&s_o[gx][d0], b1 = *(const f32x4*)&s_o[gx][d0 + 4];
#pragma unroll
    for (int e = 0; e < 4; e++) { o8[e] += f * b0[e]; o8[4 + e] += f * b1[e]; }
  }
  const float inv = 1.0f / L;
  uint32_t wv[4];
#pragma unroll
  for (int e = 0; e < 4; e++)
    wv[e] = (uint32_t)f2bf(o8[2 * e] * inv) | ((uint32_t)f2bf(o8[2 * e + 1] * inv) << 16);
  *(uint4*)(o + atile_off(mg.row, ((kvh << gshift) + hq) * 128 + d0, nq * 128)) =
      make_uint4(wv[0], wv[1], wv[2], wv[3]);
}

// Norm, RoPE and the cache write inside the decode attention: a launch less and the queries' way through memory, 1.4 to 2.9 us a layer
// where the keys and values of all rows take less time than that chain (16 heads over 8: 1 row 1.6 to 2.8 us, 16 rows over 3000 keys
// 2.9, 96 over 1000 1.4).  The more keys there are, the sooner the memory is busy all the time, and then the prologue's dependent reads
// wait behind the pages of the others.  us a layer of whole steps in favour of it, both caches, 128 / 64 / 40 rows of 32 heads over 8 and
// 128 / 64 of 16 over 8: 262 MB 0 to 3.5 (mean 1.8), 393 MB -0.4 to 1.7 (0.6), 524 MB -1.3 to 1.8 (0.4), 655 MB -3.0 to 1.9 (-0.6),
// 786 MB -5.3 to 0.5 (-1.6), 1049 MB -4.8 to 0.2 (-2.7).  40 long rows stay ahead to 786 MB, 128 short ones fall behind soon after
// 400, the last at which none loses more than two runs of one side differ.
// The prologue has lanes for ten heads: groups of up to eight queries, a key and a value.
bool attention_takes_rope(double kv_bytes, const ModelDims& md) { return md.nq / md.nkv <= 8 && kv_bytes <= 400e6; }
void launch_attention_mfma(hipStream_t s, const bf16_t* q, KvPool pool, const AttnItem* items,
                           int n_items, const AttnMerge* merges, int n_merges,
                           const int32_t* rowlist, const int32_t* page_table, bf16_t* o,
                           float* scratch, const ModelDims& md, bool prefill, const RopeArgs* rope) {
  if (n_items <= 0) return;
  float scale2 = 1.4426950408889634f / sqrtf((float)md.d);
  int gshift = 0;
  while ((1 << gshift) < md.nq / md.nkv) gshift++;
  const char* kp = (const char*)pool.k;
  const char* vp = (const char*)pool.v;
  const dim3 grid(n_items * md.nkv);
  if (prefill) {
    if (md.kv_fp8)
      attention_prefill_kernel<true><<<grid, 256, 0, s>>>(q, kp, vp, items, page_table, o, md.nq, md.nkv, gshift, md.max_pages_per_traj, scale2);
    else
      attention_prefill_kernel<false><<<grid, 256, 0, s>>>(q, kp, vp, items, page_table, o, md.nq, md.nkv, gshift, md.max_pages_per_traj, scale2);
    return;
  }
  auto go = [&](auto kernel) {
    kernel<<<grid, 256, 0, s>>>(q, (char*)pool.k, (char*)pool.v, items, rowlist, page_table, o, scratch, md.nq, md.nkv, gshift,
                                md.max_pages_per_traj, scale2, rope ? *rope : RopeArgs{});
  };
  if (md.kv_fp8) !rope ? go(attention_mfma_kernel<true, 0>) : rope->ssq ? go(attention_mfma_kernel<true, 2>) : go(attention_mfma_kernel<true, 1>);
  else !rope ? go(attention_mfma_kernel<false, 0>) : rope->ssq ? go(attention_mfma_kernel<false, 2>) : go(attention_mfma_kernel<false, 1>);
  if (n_merges > 0)
    attention_merge_kernel<<<dim3(n_merges, md.nkv), 256, 0, s>>>(scratch, merges, o, md.nq, md.nkv,
                                                                  gshift);
}
