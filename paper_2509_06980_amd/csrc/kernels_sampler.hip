// Sampling a_t ~ pi_theta(a | s_t) (paper Section 2.2) from a row of fp32 logits, bit-reproducibly.
//
// The softmax is turned into integer weights so that the cumulative sums are associative and any
// parallel reduction order gives the same token:
//   m = max z;  t_i = fl(fl(z_i - m) * c),  c = fl(log2(e) / T);
//   e_i = 2^floor(t_i) * P(t_i - floor(t_i)), P a fixed degree-6 polynomial evaluated by Horner
//   with separately rounded multiply and add; e_i = 0 below 2^-40;
//   w_i = floor(e_i * 2^32);  W = sum w_i;  r = (u32 * W) >> 32;  id = min{k : w_0+..+w_k > r}.
// The log-prob is t_id * ln 2 - ln(sum e_i).  This file must be compiled with
// -ffp-contract=off: a fused multiply-add would change the weights' bits.
//
// Launches: maxima (of segments of RL_SAMPLER_SEG logits, or of a workgroup's; left out where the lm-head has left
// maxima of its own), weight sums of the segments, then one workgroup per row that locates the segment
// and the token inside it.
#include "../../include/rl_rollout.h"
#include "kernels.h"

#include <algorithm>
#include <type_traits>

#pragma clang fp contract(off)

// x = e * 2^32 (exact scaling) and w = floor(x).  e < 1 except at the maximum, where it is exactly 1 (or
// 1 by rounding just below it), so w fits 32 bits except there: w is converted as one 32-bit integer that saturates at
// 2^32 - 1, and the caller adds the missing kTop where x >= 2^32.  A NaN gives weight 0.  The weights pass is bound by
// these instructions (128 x 151 936 logits), so none is spent twice: the polynomial's coefficients carry the 2^32 (a power
// of two changes no rounding), and both conversions are the instructions themselves, whose results beyond the integers
// are defined (saturation; zero for NaN) where C++ would need a clamp in front: rl_sample on 128 rows
// 39.7 -> 38.0 us where the last-level cache still holds the logits.  (Logits from memory: the weights pass gains as much, the
// pass for the maxima before it takes 28.8 us instead of 14.5; all three kernels 55.9 -> 53.5 us with the grid below.)
constexpr float kTwo32 = 4294967296.0f;
constexpr uint32_t kTop = 1;
__device__ __forceinline__ void exp2_weight(float z, float m, float c, float& x, uint32_t& w) {
  const float C0 = 0x1.0p32f, C1 = 0x1.62e430p31f, C2 = 0x1.ebfc40p29f, C3 = 0x1.c69f6ap27f, C4 = 0x1.3c4a8ap25f,
              C5 = 0x1.4ca4ccp22f, C6 = 0x1.b4d1e4p19f;
  float t = __fmul_rn(__fsub_rn(z, m), c);
  float n = floorf(t);
  float r = __fsub_rn(t, n);
  float p = C6;
  p = __fadd_rn(__fmul_rn(p, r), C5);
  p = __fadd_rn(__fmul_rn(p, r), C4);
  p = __fadd_rn(__fmul_rn(p, r), C3);
  p = __fadd_rn(__fmul_rn(p, r), C2);
  p = __fadd_rn(__fmul_rn(p, r), C1);
  p = __fadd_rn(__fmul_rn(p, r), C0);
  int e;
  asm("v_cvt_i32_f32 %0, %1" : "=v"(e) : "v"(n));
  x = __builtin_amdgcn_ldexpf(p, e);
  if (n < -40.0f) x = 0.f;
  asm("v_cvt_u32_f32 %0, %1" : "=v"(w) : "v"(x));
}

__host__ __device__ __forceinline__ uint32_t splitmix_u32(uint64_t seed, int32_t traj, int32_t pos) {
  uint64_t ctr = (((uint64_t)(uint32_t)traj << 32) | (uint64_t)(uint32_t)pos) + 1ull;
  uint64_t z = seed + ctr * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  return (uint32_t)(z >> 32);
}

extern "C" uint32_t rl_uniform_u32(uint64_t seed, int32_t traj_id, int32_t position) {
  return splitmix_u32(seed, traj_id, position);
}

// The 16 logits of a thread in segment `seg`: VEC (rows of whole, aligned 16-byte pieces): four pieces
// per thread, all requested before the first use; otherwise single logits.  The order of a thread's
// logits is ascending either way.
template <bool VEC>
__device__ __forceinline__ int seg_index(int seg, int tid, int i) {
  return VEC ? seg * RL_SAMPLER_SEG + ((i >> 2) * 256 + tid) * 4 + (i & 3) : seg * RL_SAMPLER_SEG + i * 256 + tid;
}
__device__ __forceinline__ bool s_whole(int seg, int V) { return (int64_t)(seg + 1) * RL_SAMPLER_SEG <= V; }
template <bool VEC>
__device__ __forceinline__ void seg_load(const float* __restrict__ zr, int V, int seg, int tid, float (&v)[16]) {
  if (VEC) {
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const int idx = seg_index<true>(seg, tid, 4 * i);
      const float4 q = *(const float4*)(zr + (idx < V ? idx : 0));
      v[4 * i] = q.x; v[4 * i + 1] = q.y; v[4 * i + 2] = q.z; v[4 * i + 3] = q.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < 16; i++) {
      const int idx = seg_index<false>(seg, tid, i);
      v[i] = zr[idx < V ? idx : 0];
    }
  }
}

// grid (nseg, rows), block 256.  Bound by the read of the logits: 14.1 us for 128 x 151 936 (5.5 TB/s;
// 22.9 us with one 4-byte read at a time).
template <bool VEC>
__global__ __launch_bounds__(256) void seg_max_kernel(const float* __restrict__ z, size_t ldz, int V,
                                                      float* __restrict__ segmax,
                                                      int32_t* __restrict__ segarg) {
  __shared__ float sv[4];
  __shared__ int si[4];
  int seg = blockIdx.x, row = blockIdx.y, nseg = gridDim.x;
  float v[16];
  seg_load<VEC>(z + (size_t)row * ldz, V, seg, threadIdx.x, v);
  float best = -INFINITY;
  int bi = 0x7fffffff;
#pragma unroll
  for (int i = 0; i < 16; i++) {
    const int idx = seg_index<VEC>(seg, threadIdx.x, i);
    if (idx < V && (v[i] > best || (v[i] == best && idx < bi))) { best = v[i]; bi = idx; }
  }
  for (int o = 32; o > 0; o >>= 1) {
    float ov = __shfl_xor(best, o, 64);
    int oi = __shfl_xor(bi, o, 64);
    if (ov > best || (ov == best && oi < bi)) { best = ov; bi = oi; }
  }
  if ((threadIdx.x & 63) == 0) { sv[threadIdx.x >> 6] = best; si[threadIdx.x >> 6] = bi; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < 4; k++)
      if (sv[k] > best || (sv[k] == best && si[k] < bi)) { best = sv[k]; bi = si[k]; }
    segmax[(size_t)row * nseg + seg] = best;
    segarg[(size_t)row * nseg + seg] = bi;
  }
}

// grid (ceil(nseg / spw), rows), block 256: the maximum of up to spw consecutive segments of a row (drawn rows: no arg-max).  The next
// segment's logits are requested before the current one's are compared: 128 x 151 936 logits 12.3 us (14.1 with a
// workgroup, its reduction and its two entries per segment, which the arg-max needs).
template <bool VEC>
__global__ __launch_bounds__(256) void row_max_kernel(const float* __restrict__ z, size_t ldz, int V, int spw, int nseg,
                                                      float* __restrict__ maxima) {
  __shared__ float sm[4];
  const int row = blockIdx.y, tid = threadIdx.x;
  const int s0 = blockIdx.x * spw, s1 = min(s0 + spw, nseg);
  const float* zr = z + (size_t)row * ldz;
  float v[16], m = -INFINITY;
  seg_load<VEC>(zr, V, s0, tid, v);
  for (int seg = s0; seg < s1; seg++) {
    float nx[16];
    if (seg + 1 < s1) seg_load<VEC>(zr, V, seg + 1, tid, nx);
#pragma unroll
    for (int i = 0; i < 16; i++) m = fmaxf(m, seg_index<VEC>(seg, tid, i) < V ? v[i] : -INFINITY);
    if (seg + 1 < s1) {
#pragma unroll
      for (int i = 0; i < 16; i++) v[i] = nx[i];
    }
  }
  m = wave_max(m);
  if ((tid & 63) == 0) sm[tid >> 6] = m;
  __syncthreads();
  if (tid == 0) maxima[(size_t)row * gridDim.x + blockIdx.x] = fmaxf(fmaxf(sm[0], sm[1]), fmaxf(sm[2], sm[3]));
}

// grid (ceil(nseg / spw), rows), block 256: weight sums of up to spw <= 8 consecutive segments of a row.
// The row maximum is first reduced from `maxima` (nmax per row: the lm-head's strip maxima, or those of the kernel
// above): several segments per workgroup, so that reading the maxima stays a small part of
// its work and needs no launch of its own.  The next segment's logits are requested before the
// current one's arithmetic.  A thread leaves its sums of a segment in LDS and goes on; behind the last one a wave adds up
// every fourth segment, so that the chains of lane exchanges and the barriers come once per workgroup and not per segment: 128 x 151 936
// logits 16.2 us (18.4 with a reduction and two barriers per segment; 30 us, and 38 + 8 us with a launch of its own for the maxima,
// before).  The integer sums take any order; a log-prob's bits are those of fp32 sums over a wave's 64 threads, halves first, and then over
// the four waves, so sixteen lanes add up one wave's (rotated in LDS so that they meet no bank twice).  put_max: the maximum is left in the row's segmax entries for the last kernel (arg-max: they hold every segment's own).
constexpr int kMaxSpw = 8;
template <bool VEC>
__global__ __launch_bounds__(256) void seg_weight_kernel(const float* __restrict__ z, size_t ldz, int V, float c,
                                                         const float* maxima, int nmax, int spw, int nseg, int put_max,
                                                         float* segmax, uint64_t* __restrict__ segw,
                                                         float* __restrict__ sege) {
  __shared__ float sm[4];
  __shared__ uint64_t sw[kMaxSpw][256];
  __shared__ float se[kMaxSpw][256];
  const int row = blockIdx.y, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int s0 = blockIdx.x * spw, s1 = min(s0 + spw, nseg);
  const float* zr = z + (size_t)row * ldz;
  float v[16];
  seg_load<VEC>(zr, V, s0, tid, v);
  float m = -INFINITY;
  const float* mr = maxima + (size_t)row * nmax;
  for (int k = tid; k < nmax; k += 256 * 8) {      // eight independent reads in flight
    float q[8];
#pragma unroll
    for (int j = 0; j < 8; j++) q[j] = mr[min(k + 256 * j, nmax - 1)];
#pragma unroll
    for (int j = 0; j < 8; j++) m = fmaxf(m, q[j]);
  }
  m = wave_max(m);
  if (lane == 0) sm[wave] = m;
  __syncthreads();
  m = fmaxf(fmaxf(sm[0], sm[1]), fmaxf(sm[2], sm[3]));
  for (int seg = s0; seg < s1; seg++) {
    float nx[16];
    if (seg + 1 < s1) seg_load<VEC>(zr, V, seg + 1, tid, nx);
    uint64_t ws = 0;
    float es = 0.f;
    float xm = 0.f;
    if (s_whole(seg, V)) {              // no element of the segment lies behind the row's end
      float xs[16];
#pragma unroll
      for (int i = 0; i < 16; i++) {
        float x;
        uint32_t w;
        exp2_weight(v[i], m, c, x, w);
        ws += w;
        es = __fadd_rn(es, x);
        xs[i] = x;
      }
#pragma unroll
      for (int i = 0; i < 16; i += 2) xm = fmaxf(fmaxf(xm, xs[i]), xs[i + 1]);      // one instruction for two
    } else {
#pragma unroll
      for (int i = 0; i < 16; i++) {
        float x;
        uint32_t w;
        exp2_weight(v[i], m, c, x, w);
        const bool in = seg_index<VEC>(seg, tid, i) < V;
        ws += in ? w : 0u;
        es = __fadd_rn(es, in ? x : 0.f);
        xm = in ? fmaxf(xm, x) : xm;
      }
    }
    if (__any(xm >= kTwo32)) {          // the row's maximum is among the wave's elements
#pragma unroll
      for (int i = 0; i < 16; i++) {
        float x;
        uint32_t w;
        exp2_weight(v[i], m, c, x, w);
        if (x >= kTwo32 && seg_index<VEC>(seg, tid, i) < V) ws += kTop;
      }
    }
    sw[seg - s0][tid] = ws;
    se[seg - s0][tid ^ wave << 4] = es;
    if (seg + 1 < s1) {
#pragma unroll
      for (int i = 0; i < 16; i++) v[i] = nx[i];
    }
  }
  __syncthreads();
  for (int seg = s0 + wave; seg < s1; seg += 4) {
    const uint64_t* pw = sw[seg - s0] + lane;
    uint64_t ws = (pw[0] + pw[64]) + (pw[128] + pw[192]);
    const int w = lane >> 4;
    const float* pe = se[seg - s0] + w * 64;
    auto of = [&](int t) { return pe[t ^ w << 4]; };      // thread t of wave w
    float es = __fadd_rn(__fadd_rn(of(lane & 15), of((lane & 15) + 32)), __fadd_rn(of((lane & 15) + 16), of((lane & 15) + 48)));
#pragma unroll
    for (int k = 0; k < 6; k++) {
      ws += __shfl_xor(ws, 1 << k, 64);
      es = __fadd_rn(es, __shfl_xor(es, k < 4 ? 8 >> k : 1 << k, 64));
    }
    if (lane == 0) {
      segw[(size_t)row * nseg + seg] = ws;
      sege[(size_t)row * nseg + seg] = es * 0x1p-32f;
      if (put_max) segmax[(size_t)row * nseg + seg] = m;
    }
  }
}

// Sums over a wave's lanes up to and including this one.
__device__ __forceinline__ uint64_t wave_scan(uint64_t x) {
  const int lane = threadIdx.x & 63;
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  return x;
}

// Inclusive sum over the workgroup's threads; *total gets the sum of all.  tmp: an entry of LDS per wave.
__device__ __forceinline__ uint64_t block_scan(uint64_t x, uint64_t* tmp, int waves, uint64_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  x = wave_scan(x);
  __syncthreads();                      // an earlier use of tmp is over
  if (lane == 63) tmp[wave] = x;
  __syncthreads();
  uint64_t before = 0, all = 0;
  for (int k = 0; k < waves; k++) {
    const uint64_t y = tmp[k];
    before += k < wave ? y : 0;
    all += y;
  }
  *total = all;
  return x + before;
}

// grid rows, block 256.  A chain of two dependent reads (segment sums and the draw; the chosen segment's logits).  FEW (at most 64
// segments): every wave holds all segments, one a lane, and finds the segment by itself; the only barriers are those of the
// search among the segment's logits (1 / 128 rows of 151 936 logits 5.4 / 6.7 us with the segments joined through LDS and the draw read
// behind their sums, now 4.8 / 5.8; 1024 threads of four logits 5.5 / 6.3; 15.1 with one thread's loops).
template <bool VEC, bool FEW>
__global__ __launch_bounds__(256) void sample_final_kernel(
    const float* __restrict__ z, size_t ldz, int V, float c, int greedy, int nseg,
    const float* __restrict__ segmax, const int32_t* __restrict__ segarg, const uint64_t* __restrict__ segw,
    const float* __restrict__ sege, const uint32_t* __restrict__ u32, uint64_t seed,
    const int32_t* __restrict__ row_traj, const int32_t* __restrict__ row_newpos,
    const int32_t* __restrict__ forced, const uint8_t* __restrict__ out_mask, int32_t* __restrict__ ids_out,
    float* __restrict__ logp_out) {
  constexpr int T = 256, NW = T / 64, PER = RL_SAMPLER_SEG / T;      // consecutive logits per thread
  __shared__ uint64_t tmp[NW], s_pre;
  __shared__ float sm[NW], se[NW], s_z;
  __shared__ int sa[NW], s_seg, s_id;
  const int row = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const float* zr = z + (size_t)row * ldz;
  const size_t r0 = (size_t)row * nseg;
  const bool drawn = !(forced || greedy);
  // asked for ahead of the sums that they are used behind
  const int want = forced ? forced[row] : 0;
  const uint32_t u = !drawn ? 0u : u32 ? u32[row] : splitmix_u32(seed, row_traj[row], row_newpos[row]);
  const bool masked = out_mask && out_mask[row];
  float m = -INFINITY, E = 0.f;
  int arg = 0x7fffffff;
  uint64_t W = 0, own = 0;
  for (int k = FEW ? lane : tid; k < nseg; k += FEW ? 64 : T) {
    const float v = segmax[r0 + k];
    if (greedy) {
      const int a = segarg[r0 + k];
      if (v > m || (v == m && a < arg)) { m = v; arg = a; }
    } else {
      m = fmaxf(m, v);
    }
    own = segw[r0 + k];
    W += own;
    E = __fadd_rn(E, sege[r0 + k]);
  }
  if (tid == 0) { s_seg = nseg - 1; s_id = -1; }
  const uint64_t incl = FEW ? wave_scan(W) : 0;
  for (int o = 32; o > 0; o >>= 1) {
    const float ov = __shfl_xor(m, o, 64);
    const int oa = __shfl_xor(arg, o, 64);
    if (greedy ? (ov > m || (ov == m && oa < arg)) : ov > m) { m = ov; arg = oa; }
    E = __fadd_rn(E, __shfl_xor(E, o, 64));
    if (!FEW) W += __shfl_xor(W, o, 64);
  }
  if (FEW) {
    W = __shfl(incl, 63, 64);
  } else {
    if (lane == 0) { sm[wave] = m; sa[wave] = arg; se[wave] = E; tmp[wave] = W; }
    __syncthreads();
    m = sm[0];
    arg = sa[0];
    for (int k = 1; k < NW; k++)
      if (sm[k] > m || (sm[k] == m && sa[k] < arg)) { m = sm[k]; arg = sa[k]; }
    E = __fadd_rn(__fadd_rn(se[0], se[1]), __fadd_rn(se[2], se[3]));
    W = tmp[0] + tmp[1] + tmp[2] + tmp[3];
  }
  int id;
  float zid = 0.f;
  if (!drawn) {
    id = forced ? want : (arg == 0x7fffffff ? 0 : arg);   // a row without any number: token 0
    if (id >= 0 && id < V) zid = zr[id];
  } else {
    const uint64_t hi = __umul64hi(W, (uint64_t)u), lo = W * (uint64_t)u;
    const uint64_t r = (hi << 32) | (lo >> 32);          // floor(u * W / 2^32) < W
    // first segment whose inclusive sum exceeds r (the last one if none does)
    int s;
    uint64_t rl;                                         // target inside segment s
    if (FEW) {
      const uint64_t above = __ballot(lane < nseg - 1 && incl > r);
      s = above ? __builtin_ctzll(above) : nseg - 1;
      rl = r - (__shfl(incl, s, 64) - __shfl(own, s, 64));
    } else {
      uint64_t carry = 0;
      for (int k0 = 0; k0 < nseg; k0 += T) {
        const int k = k0 + tid;
        const uint64_t w = k < nseg ? segw[r0 + k] : 0;
        uint64_t total;
        const uint64_t in = carry + block_scan(w, tmp, NW, &total);
        if (k < nseg - 1 && in > r && in - w <= r) { s_seg = k; s_pre = in - w; }
        if (k == nseg - 1 && in - w <= r) s_pre = in - w;
        carry += total;
      }
      __syncthreads();
      s = s_seg;
      rl = r - s_pre;
    }
    const int base = s * RL_SAMPLER_SEG + tid * PER;
    float zl[PER];
    if (VEC) {
#pragma unroll
      for (int j = 0; j < PER; j += 4) {
        const float4 q = *(const float4*)(zr + (base + j < V ? base + j : 0));
        zl[j] = q.x; zl[j + 1] = q.y; zl[j + 2] = q.z; zl[j + 3] = q.w;
      }
    } else {
#pragma unroll
      for (int j = 0; j < PER; j++) zl[j] = zr[base + j < V ? base + j : 0];
    }
    uint64_t wloc[PER];
    uint64_t mine = 0;
#pragma unroll
    for (int j = 0; j < PER; j++) {
      float x;
      uint32_t w;
      exp2_weight(zl[j], m, c, x, w);
      wloc[j] = base + j < V ? (uint64_t)w + (x >= kTwo32 ? kTop : 0u) : 0;
      mine += wloc[j];
    }
    uint64_t total;
    const uint64_t before = block_scan(mine, tmp, NW, &total) - mine;
    if (before <= rl && rl < before + mine) {
      uint64_t acc = before;
      bool found = false;
#pragma unroll
      for (int j = 0; j < PER; j++) {
        acc += wloc[j];
        if (!found && acc > rl) { found = true; s_id = base + j; s_z = zl[j]; }
      }
    }
    __syncthreads();
    // no weight at all (a row of NaN, or one with plus infinity): token 0 and no number as its log-prob.  The
    // id has to lie in the vocabulary: a decode step embeds it
    id = s_id < 0 ? 0 : s_id;
    zid = s_id < 0 ? __builtin_nanf("") : s_z;
  }
  if (tid == 0) {
    float lp = 0.f;
    if (!masked) {
      float t = __fmul_rn(__fsub_rn(zid, m), c);
      lp = t * 0.6931471805599453f - logf(E);
    }
    if (ids_out) ids_out[row] = id;
    logp_out[row] = lp;
  }
}

// Where the line lies: rl_sample on 1 / 256 rows of 4096 logits 12.8 / 14.8 -> 5.3 / 6.1 us, 8192 13.4 / 15.5 -> 6.1 / 7.2,
// 16384 13.3 / 17.9 -> 9.1 / 10.6.  A thread holds no more than 16, and rows that cannot be read in 16-byte pieces lose from
// 8192 on (16001, greedy: 11.3 -> 13.5).
constexpr int kRowLogits = 16384, kRowLogitsScalar = 4096;
// Rows of up to 16 T logits: maximum, weights, sums and search in one workgroup of T threads, 16 consecutive logits a
// thread, all in registers.  The three launches above are three latency chains (4 rows of 4096: 3.5 + 4.4 + 3.4 us and the gaps
// between them); a row that fits one workgroup needs none of their hand-over through memory.
template <int T, bool VEC>
__global__ __launch_bounds__(T) void sample_row_kernel(
    const float* __restrict__ z, size_t ldz, int V, float c, int greedy, const uint32_t* __restrict__ u32, uint64_t seed,
    const int32_t* __restrict__ row_traj, const int32_t* __restrict__ row_newpos, const int32_t* __restrict__ forced,
    const uint8_t* __restrict__ out_mask, int32_t* __restrict__ ids_out, float* __restrict__ logp_out) {
  constexpr int NW = T / 64, PER = 16;
  __shared__ float sm[NW], se[NW], s_z;
  __shared__ int sa[NW], s_id;
  __shared__ uint64_t sw[NW];
  const int row = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, base = tid * PER;
  const float* zr = z + (size_t)row * ldz;
  float v[PER];
  if (VEC) {
#pragma unroll
    for (int j = 0; j < PER; j += 4) {
      const float4 q = *(const float4*)(zr + (base + j < V ? base + j : 0));
      v[j] = q.x; v[j + 1] = q.y; v[j + 2] = q.z; v[j + 3] = q.w;
    }
  } else {
#pragma unroll
    for (int j = 0; j < PER; j++) v[j] = zr[base + j < V ? base + j : 0];
  }
  const int want = forced ? forced[row] : -1;
  float m = -INFINITY;
  int arg = 0x7fffffff;
#pragma unroll
  for (int j = 0; j < PER; j++)
    if (base + j < V && (v[j] > m || (v[j] == m && base + j < arg))) { m = v[j]; arg = base + j; }
  for (int o = 32; o > 0; o >>= 1) {
    const float ov = __shfl_xor(m, o, 64);
    const int oa = __shfl_xor(arg, o, 64);
    if (ov > m || (ov == m && oa < arg)) { m = ov; arg = oa; }
  }
  if (lane == 0) { sm[wave] = m; sa[wave] = arg; }
  if (tid == 0) { s_id = -1; s_z = 0.f; }
  __syncthreads();
  m = sm[0];
  arg = sa[0];
  for (int k = 1; k < NW; k++)
    if (sm[k] > m || (sm[k] == m && sa[k] < arg)) { m = sm[k]; arg = sa[k]; }
  // 1024 threads have 128 registers each, which sixteen 64-bit weights leave no room in (12 bytes of scratch a lane): they hold the
  // conversion saturated at 2^32 - 1, to which no float below 2^32 converts, and the search forms the weights again (64 rows
  // of 16384 logits 10.3 -> 9.9 us; with 256 and 512 threads, which have the room, the drawn rows took 0.2 to 0.3 us more).
  constexpr bool SAT = T == 1024;
  std::conditional_t<SAT, uint32_t, uint64_t> wl[PER];
  auto weight = [&](int j) { return SAT ? (uint64_t)wl[j] + (wl[j] == 0xffffffffu ? kTop : 0u) : (uint64_t)wl[j]; };
  uint64_t mine = 0;
  float e = 0.f;
#pragma unroll
  for (int j = 0; j < PER; j++) {
    float x;
    uint32_t w;
    exp2_weight(v[j], m, c, x, w);
    const bool in = base + j < V;
    if constexpr (SAT) {
      wl[j] = in ? w : 0u;
      mine += weight(j);
      asm volatile("" : "+v"(wl[j]));      // or the 64-bit weights would be kept after all
    } else {
      wl[j] = in ? (uint64_t)w + (x >= kTwo32 ? kTop : 0u) : 0;
      mine += wl[j];
    }
    e = __fadd_rn(e, in ? x : 0.f);
  }
  const uint64_t incl = wave_scan(mine);
  for (int o = 32; o > 0; o >>= 1) e = __fadd_rn(e, __shfl_xor(e, o, 64));
  if (lane == 63) sw[wave] = incl;
  if (lane == 0) se[wave] = e;
  __syncthreads();
  uint64_t before = incl - mine, W = 0;
  float E = 0.f;
  for (int k = 0; k < NW; k++) {
    if (k < wave) before += sw[k];
    W += sw[k];
    E = __fadd_rn(E, se[k]);
  }
  E *= 0x1p-32f;
  if (forced || greedy) {
    const int id = forced ? want : (arg == 0x7fffffff ? 0 : arg);      // a row without any number: token 0
#pragma unroll
    for (int j = 0; j < PER; j++)
      if (base + j == id && id < V) s_z = v[j];
    if (tid == 0) s_id = id;
  } else {
    const uint32_t u = u32 ? u32[row] : splitmix_u32(seed, row_traj[row], row_newpos[row]);
    const uint64_t hi = __umul64hi(W, (uint64_t)u), lo = W * (uint64_t)u;
    const uint64_t r = (hi << 32) | (lo >> 32);          // floor(u * W / 2^32) < W
    if (before <= r && r < before + mine) {
      uint64_t acc = before;
      bool found = false;
#pragma unroll
      for (int j = 0; j < PER; j++) {
        acc += weight(j);
        if (!found && acc > r) { found = true; s_id = base + j; s_z = v[j]; }
      }
    }
  }
  __syncthreads();
  if (tid == 0) {
    const bool drawn = !(forced || greedy);
    const int id = drawn && s_id < 0 ? 0 : s_id;         // no weight at all: token 0 and no number as its log-prob
    const float zid = drawn && s_id < 0 ? __builtin_nanf("") : s_z;
    float lp = 0.f;
    if (!(out_mask && out_mask[row])) lp = __fmul_rn(__fsub_rn(zid, m), c) * 0.6931471805599453f - logf(E);
    if (ids_out) ids_out[row] = id;
    logp_out[row] = lp;
  }
}

static bool whole_pieces(const float* logits, size_t ldz, int V) {
  return V % 4 == 0 && ldz % 4 == 0 && ((uintptr_t)logits & 15) == 0;
}
static bool row_in_one_workgroup(bool vec, int V) { return V <= (vec ? kRowLogits : kRowLogitsScalar); }
bool sampler_reads_maxima(const float* logits, size_t ldz, int V, bool greedy) {
  return !greedy && !row_in_one_workgroup(whole_pieces(logits, ldz, V), V);
}
void launch_sampler(hipStream_t s, const float* logits, size_t ldz, int rows, int V, float scale_c,
                    int greedy, const uint32_t* u32, uint64_t seed, const int32_t* row_traj,
                    const int32_t* row_newpos, const int32_t* forced, const uint8_t* out_mask,
                    SamplerScratch sc, int32_t* ids_out, float* logp_out, const float* stripmax,
                    int nstrips) {
  if (rows <= 0) return;
  const int nseg = sampler_nseg(V);
  const dim3 grid(nseg, rows);
  const bool vec = whole_pieces(logits, ldz, V);
  if (row_in_one_workgroup(vec, V)) {
    auto go = [&](auto kernel, int threads) {
      kernel<<<rows, threads, 0, s>>>(logits, ldz, V, scale_c, greedy, u32, seed, row_traj, row_newpos, forced, out_mask, ids_out, logp_out);
    };
    static_assert(kRowLogitsScalar <= 16 * 256, "the scalar form has 256 threads");
    if (V <= 16 * 256) vec ? go(sample_row_kernel<256, true>, 256) : go(sample_row_kernel<256, false>, 256);
    else if (V <= 8192) go(sample_row_kernel<512, true>, 512);
    else go(sample_row_kernel<1024, true>, 1024);
    return;
  }
  if (greedy || nstrips <= 0) stripmax = nullptr;   // the arg-max needs the pass over the logits
  // about five workgroups per CU, each with at most eight segments (rl_sample on 128 rows of 151936 / 40000 logits: four 38.0 /
  // 20.8 us, five 37.7 / 18.5, eight 38.9 / 18.6)
  const int spw = (int)std::min<int64_t>(kMaxSpw, std::max<int64_t>(1, ((int64_t)nseg * rows + 1279) / 1280));
  const dim3 wgrid((nseg + spw - 1) / spw, rows);
  // of drawn rows the workgroups' maxima go where the arg-max would: the weights' kernel writes segmax while others still read
  const float* maxima = stripmax ? stripmax : greedy ? sc.segmax : (const float*)sc.segarg;
  const int nmax = stripmax ? nstrips : greedy ? nseg : (int)wgrid.x;
  auto go = [&](auto vec_) {
    constexpr bool VEC = decltype(vec_)::value;
    if (greedy) seg_max_kernel<VEC><<<grid, 256, 0, s>>>(logits, ldz, V, sc.segmax, sc.segarg);
    else if (!stripmax) row_max_kernel<VEC><<<wgrid, 256, 0, s>>>(logits, ldz, V, spw, nseg, (float*)sc.segarg);
    seg_weight_kernel<VEC><<<wgrid, 256, 0, s>>>(logits, ldz, V, scale_c, maxima, nmax, spw, nseg, greedy ? 0 : 1, sc.segmax, sc.segw, sc.sege);
    auto last = [&](auto kernel) {
      kernel<<<rows, 256, 0, s>>>(logits, ldz, V, scale_c, greedy, nseg, sc.segmax, sc.segarg, sc.segw, sc.sege, u32, seed, row_traj, row_newpos,
                                  forced, out_mask, ids_out, logp_out);
    };
    if (nseg <= 64) last(sample_final_kernel<VEC, true>);
    else last(sample_final_kernel<VEC, false>);
  };
  if (vec) go(std::true_type());
  else go(std::false_type());
}

// ---------------------------------------------------------------------------------------------
// The sampler for callers that must not allocate device memory.  Its per-segment scratch lives in
// a fixed array in the library's device image; every GPU holds its own copy at its own address,
// looked up once per device.  Host code uses that address only, never the array's name.
// ---------------------------------------------------------------------------------------------
#define RL_NOALLOC_MAX_SEGMENTS 16384   // rows x ceil(vocab / RL_SAMPLER_SEG) of one call
#define RL_NOALLOC_SEG_BYTES 24         // max 4 + arg 4 + weight 8 + sum 4, padded to keep 8-byte alignment
static __device__ __align__(256) unsigned char scratch[(size_t)RL_NOALLOC_MAX_SEGMENTS * RL_NOALLOC_SEG_BYTES];

#define RL_MAX_DEVICES 64
static unsigned char* g_scratch_ptr[RL_MAX_DEVICES];   // per device: address of its copy of `scratch`

// Address of the current device's scratch array (looked up on first use), or null with *err set.
static unsigned char* noalloc_scratch(hipError_t* err) {
  int dev = 0;
  *err = hipGetDevice(&dev);
  if (*err != hipSuccess) return nullptr;
  if (dev < 0 || dev >= RL_MAX_DEVICES) { *err = hipErrorInvalidDevice; return nullptr; }
  if (!g_scratch_ptr[dev]) {
    unsigned char* p = nullptr;
    *err = hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch));
    if (*err != hipSuccess) return nullptr;
    g_scratch_ptr[dev] = p;
  }
  return g_scratch_ptr[dev];
}

int sampler_noalloc_prepare() {
  hipError_t e;
  return noalloc_scratch(&e) ? 0 : (int)e;
}

extern "C" int rl_sample_device_logits(const float* d_logits, int32_t rows, int32_t vocab,
                                       float temperature, const uint32_t* d_u32, int32_t* d_ids_out,
                                       float* d_logprobs_out, void* stream) {
  if (!d_logits || !d_u32 || !d_ids_out || !d_logprobs_out || rows <= 0 || vocab <= 0 ||
      !(temperature >= 0.0f))
    return rl_fail(RL_E_ARG, "bad argument");
  const int nseg = sampler_nseg(vocab);
  const size_t seg_n = (size_t)rows * nseg;
  if (seg_n > RL_NOALLOC_MAX_SEGMENTS)
    return rl_fail(RL_E_ARG, "rows x ceil(vocab / 4096) exceeds the 16384 segments of the fixed scratch");
  hipError_t e;
  unsigned char* base = noalloc_scratch(&e);
  if (!base) return rl_fail(RL_E_HIP, hipGetErrorString(e));
  // every entry the final kernel reads is written by the two segment kernels of this call first:
  // nothing has to start at zero
  SamplerScratch sc;
  sc.segw = (uint64_t*)base;
  sc.segmax = (float*)(sc.segw + seg_n);
  sc.segarg = (int32_t*)(sc.segmax + seg_n);
  sc.sege = (float*)(sc.segarg + seg_n);
  const bool greedy = temperature == 0.0f;
  const float c = sampler_scale(temperature);
  launch_sampler((hipStream_t)stream, d_logits, (size_t)vocab, rows, vocab, c, greedy ? 1 : 0, d_u32, 0,
                 nullptr, nullptr, nullptr, nullptr, sc, d_ids_out, d_logprobs_out);
  e = hipGetLastError();
  if (e != hipSuccess) return rl_fail(RL_E_HIP, hipGetErrorString(e));
  return RL_OK;
}
