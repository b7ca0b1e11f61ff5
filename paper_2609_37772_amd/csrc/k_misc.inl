// Per-token kernels of the step: the per-token time embedding and action
// input projection, and the final norm + action projection fused with the
// masked per-token Euler update.
#include "uad_internal.h"

namespace uad {


// Sum over a 256-thread block in a fixed order (wave shuffles, then 4 partials).
__device__ __forceinline__ float block_sum_256(float v, float *scratch) {
  v = sum_wave64(v);
  const int wave = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) scratch[wave] = v;
  __syncthreads();
  return (scratch[0] + scratch[1]) + (scratch[2] + scratch[3]);
}

// Rows per workgroup of the embedding kernels: R tokens share one read of
// their columns' W_in rows (R = 16 when batched: with one token per
// workgroup the 3,200-token fleet re-read W_in 3,200 times from L2).
// Token m of a compacted step is token env_map[m / chunk] * chunk + m % chunk
// of the caller's arrays (null map: token m).
__device__ __forceinline__ int phys_token(const int32_t *env_map, int chunk, int m) {
  if (!env_map) return m;
  const int b = m / chunk;
  return env_map[b] * chunk + (m - b * chunk);
}

template <int R>
__device__ __forceinline__ int load_action_rows(const float *__restrict__ x, int M, int Da, float (*xs)[64],
                                                const int32_t *env_map = nullptr, int chunk = 1) {
  const int m0 = blockIdx.x * R;
  const int rows = min(R, M - m0);
  for (int i = threadIdx.x; i < rows * Da; i += blockDim.x) {
    const int r = i / Da, j = i - r * Da;
    xs[r][j] = x[(size_t)phys_token(env_map, chunk, m0 + r) * Da + j];
  }
  __syncthreads();
  return rows;
}

// acc[r] += sum_j xs[r][j] w[j] over one W_in row (this thread's output
// column), in j order.  16-byte loads when the row allows: each of a wave's
// load instructions then touches every lane's 128-byte row once, where
// 4-byte loads touched 64 rows per instruction 32 times over.
template <int R>
__device__ __forceinline__ void action_row_dot(const float *__restrict__ w, int Da, const float (*xs)[64],
                                               float (&acc)[R]) {
  if ((Da & 3) == 0 && ((uintptr_t)w & 15) == 0) {
    for (int j = 0; j < Da; j += 4) {
      const f32x4 w4 = *(const f32x4 *)(w + j);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r] += xs[r][j + e] * w4[e];  // rows past the end: never stored
    }
  } else {
    for (int j = 0; j < Da; ++j) {
      const float wj = w[j];
#pragma unroll
      for (int r = 0; r < R; ++r) acc[r] += xs[r][j] * wj;
    }
  }
}

// te[m] = [ x_m W_in^T + b_in ; sin(w t_m) ; cos(w t_m) ] as the fp16 operand
// of the time MLP in fragment order (K = 2d): the per-token flow-time
// conditioning placed before the action MLP.  Workgroup (g, y): tokens
// g R .. g R + R - 1, columns y * blockDim.x + tid of the action projection
// and the same indices of the sinusoids.
template <int R>
__global__ __launch_bounds__(256) void temb_kernel(const float *__restrict__ x, const float *__restrict__ t, int M,
                                                    int Da, int d, const float *__restrict__ w_in,
                                                    const float *__restrict__ b_in,
                                                    const float *__restrict__ freqs, op_t *__restrict__ te,
                                                    unsigned *status, const int32_t *env_map, int chunk) {
  __shared__ float xs[R][64];
  const int m0 = blockIdx.x * R;
  const int rows = load_action_rows<R>(x, M, Da, xs, env_map, chunk);
  const int KB = 2 * d / kTileK;
  unsigned bad = 0;  // fp16 range flag of this thread's stores
  const int n = blockIdx.y * blockDim.x + threadIdx.x;
  if (n < d) {
    float acc[R];
    const float bn = b_in[n];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = bn;
    action_row_dot<R>(w_in + (size_t)n * Da, Da, xs, acc);
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (r < rows) store_op(te + afrag_index(m0 + r, n, KB), acc[r], bad);
  }
  const int half = d >> 1;
  if (n < half)
    for (int r = 0; r < rows; ++r) {
      const float arg = freqs[n] * t[phys_token(env_map, chunk, m0 + r)];
      float sv, cv;
      sincosf(arg, &sv, &cv);  // one range reduction for both
      store_op(te + afrag_index(m0 + r, d + n, KB), sv, bad);
      store_op(te + afrag_index(m0 + r, d + half + n, KB), cv, bad);
    }
  flush_range(status, bad);
}

// Adaptive-norm variant: te[m] = e(t_m) alone (K = d) as the time MLP's fp16
// operand; the action token itself starts the residual stream,
// h[m] = x_m W_in^T + b_in (fp32), with its per-16-column sums of squares.
// t null: no time features (the schedule computed its time conditioning up
// front); mod_a0 not null: also the first attention norm's operand
// next = fp16(h_0 (1 + a)) with a the token's layer-0 scale, row stride mod_ld.
template <int R>
__global__ __launch_bounds__(256) void temb_ada_kernel(const float *__restrict__ x, const float *__restrict__ t,
                                                        int M, int Da, int d, const float *__restrict__ w_in,
                                                        const float *__restrict__ b_in,
                                                        const float *__restrict__ freqs, op_t *__restrict__ te,
                                                        float *__restrict__ h, float *__restrict__ ssq,
                                                        int m_alloc, const float *__restrict__ mod_a0, int mod_ld,
                                                        op_t *__restrict__ next, unsigned *status) {
  __shared__ float xs[R][64];
  const int m0 = blockIdx.x * R;
  const int rows = load_action_rows<R>(x, M, Da, xs);
  const int KB = d / kTileK;
  unsigned bad = 0;  // fp16 range flag of this thread's stores
  // d is a multiple of 32, so the 16 lanes of a 16-column tile are active together
  const int n = blockIdx.y * blockDim.x + threadIdx.x;
  if (n < d) {
    float acc[R];
    const float bn = b_in[n];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = bn;
    action_row_dot<R>(w_in + (size_t)n * Da, Da, xs, acc);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (r < rows) {  // uniform over the workgroup
        const int m = m0 + r;
        h[(size_t)m * d + n] = acc[r];
        float sq = acc[r] * acc[r];
        sq = sum_row16(sq);
        if ((n & 15) == 0) ssq[(size_t)(n >> 4) * m_alloc + m] = sq;
        if (mod_a0) store_op(next + afrag_index(m, n, KB), acc[r] * (1.0f + mod_a0[(size_t)m * mod_ld + n]), bad);
      }
    }
  }
  const int half = d >> 1;
  if (t && n < half)
    for (int r = 0; r < rows; ++r) {
      const float arg = freqs[n] * t[m0 + r];
      float sv, cv;
      sincosf(arg, &sv, &cv);  // one range reduction for both
      store_op(te + afrag_index(m0 + r, n, KB), sv, bad);
      store_op(te + afrag_index(m0 + r, half + n, KB), cv, bad);
    }
  flush_range(status, bad);
}

// v = RMSNorm(h) W_out^T + b_out, then x <- x + dt v unless frozen (mask or
// dt == 0: copy, so frozen tokens are bit-identical whatever v holds).
// Workgroup = (token m, group of up to 8 action dims); thread t owns columns
// t + 256 i of the row for all 8 dims, loads unconditional as above.
constexpr int kFinalOuts = 8;

// Masked Euler update of token m, action dim a with velocity v (a copy when
// frozen), the velocity outputs and the release bookkeeping.
__device__ __forceinline__ void euler_out(const FinalArgs &f, int mc, int a, float v) {
  const int m = phys_token(f.env_map, f.chunk, mc);  // the caller's token of step row mc
  const size_t idx = (size_t)m * f.Da + a;
  const float dtm = f.dt[m];
  const bool frozen = (f.mask[m] != 0) || (dtm == 0.0f);
  const float xo = f.x[idx];
  const float xn = frozen ? xo : xo + dtm * v;
  f.x[idx] = xn;
  if (f.v_out) f.v_out[idx] = v;
  if (f.vsum && (m % f.chunk) < f.vsum_tokens) f.vsum[idx] += v;
  const bool releasing = !frozen && (f.is_last_step || (f.next_mask && f.next_mask[m] != 0));
  if (releasing) {
    if (f.released) f.released[idx] = xn;
    if (f.release_step && a == 0) f.release_step[m] = f.step;
  }
}

template <int NC, bool MAP>
__global__ __launch_bounds__(256) void final_kernel(FinalArgs f) {
  __shared__ float scratch[4];
  __shared__ float wsum[4][kFinalOuts];
  __shared__ float vs[kFinalOuts];
  const int32_t *mod_row = f.mod_row;
  if (MAP) f.env_map = nullptr;
  const int m = blockIdx.x;
  const int a0 = blockIdx.y * kFinalOuts;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int d = f.d;
  if (f.debug_field) {
    if (threadIdx.x < kFinalOuts && a0 + threadIdx.x < f.Da)
      vs[threadIdx.x] = f.dbg_alpha * f.x[(size_t)phys_token(f.env_map, f.chunk, m) * f.Da + a0 + threadIdx.x] +
                        f.dbg_beta;
  } else {
    const float *__restrict__ hr = f.h + (size_t)m * d;
    float hv[NC], gv[NC], sv[NC], wv[kFinalOuts][NC];
    const bool ada = f.mod_scale != nullptr;
    const size_t mrow = (size_t)(MAP ? mod_row[m] : m) * f.mod_ld;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int c = min(threadIdx.x + 256 * i, d - 1);
      hv[i] = hr[c];
      // adaptive norm: per-token scale (1 + a) and shift b; else the gain
      gv[i] = ada ? 1.0f + f.mod_scale[mrow + c] : f.gain[c];
      sv[i] = ada ? f.mod_shift[mrow + c] : 0.f;
#pragma unroll
      for (int o = 0; o < kFinalOuts; ++o) wv[o][i] = f.w_out[(size_t)min(a0 + o, f.Da - 1) * d + c];
    }
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      if (threadIdx.x + 256 * i >= d) hv[i] = sv[i] = 0.f;  // clamped duplicate columns contribute nothing
      ss += hv[i] * hv[i];
    }
    ss = block_sum_256(ss, scratch);
    const float rstd = 1.0f / sqrtf(ss / (float)d + f.eps);
    float acc[kFinalOuts];
#pragma unroll
    for (int o = 0; o < kFinalOuts; ++o) {
      acc[o] = 0.f;
#pragma unroll
      for (int i = 0; i < NC; ++i) acc[o] += (hv[i] * rstd * gv[i] + sv[i]) * wv[o][i];
      acc[o] = sum_wave64(acc[o]);
    }
    if (lane == 0)
#pragma unroll
      for (int o = 0; o < kFinalOuts; ++o) wsum[wave][o] = acc[o];
    __syncthreads();
    if (threadIdx.x < kFinalOuts && a0 + threadIdx.x < f.Da) {
      const int o = threadIdx.x;
      vs[o] = ((wsum[0][o] + wsum[1][o]) + (wsum[2][o] + wsum[3][o])) + f.b_out[a0 + o];
    }
  }
  __syncthreads();
  if (threadIdx.x < kFinalOuts && a0 + threadIdx.x < f.Da) euler_out(f, m, a0 + threadIdx.x, vs[threadIdx.x]);
}

// Batched steps (many tokens, no debug field): the
// projection as a product on the fp32 MFMA (v_mfma_f32_16x16x4_f32), 16
// tokens x all Da outputs per workgroup, the d columns split over its 4
// waves: v = rstd * ((h * gain) W_out^T) + b_out.  The row-blocked form it
// replaces spent its time in 72 wave reductions per wave (one per token and
// output) and re-read h once per group of 8 outputs.  Within a wave, k-step
// (q, e) of lane group kq = lane / 16 covers column c0 + 16 q + 4 kq + e, so
// each lane reads 16-byte runs of h, gain and W_out and feeds the same
// column to both operands.  The k-groups run in batches of 8 (uniform trip
// count: the loop bound does not depend on kq), loads first.
// ADA: the gain is the token's 1 + scale and its shift enters through a second
// accumulator, v = rstd * ((h (1 + a)) W_out^T) + b W_out^T + b_out.
template <int NT, bool ADA>
__global__ __launch_bounds__(256) void final_mfma_kernel(FinalArgs f) {
  __shared__ f32x4 part[4][NT][64];  // per wave and output tile: each lane's accumulators
  __shared__ f32x4 part2[ADA ? 4 : 1][ADA ? NT : 1][64];  // ... of the shift
  __shared__ float ssq[4][64];       // per wave and lane: partial sum of squares of the lane's row
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m0 = blockIdx.x * 16, kq = lane >> 4;
  const float *__restrict__ hr = f.h + (size_t)min(m0 + (lane & 15), f.M - 1) * f.d;  // rows past M: never stored
  const float *__restrict__ wr[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) wr[t] = f.w_out + (size_t)min(16 * t + (lane & 15), f.Da - 1) * f.d;
  const int cpw = f.d >> 2;  // columns per wave (d % 512 == 0: whole batches)
  f32x4 acc[NT], acc2[ADA ? NT : 1];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < (ADA ? NT : 1); ++t) acc2[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float *gr = f.gain, *sr = nullptr;
  if constexpr (ADA) {
    const int mc = min(m0 + (lane & 15), f.M - 1);
    const size_t mr = (size_t)f.mod_row[mc] * f.mod_ld;  // from 1024 rows on always by class
    f.env_map = nullptr;
    gr = f.mod_scale + mr;
    sr = f.mod_shift + mr;
  }
  float ss = 0.f;
  // batches of 8 k-groups of 16 columns: all their loads go out before the first MFMA
  for (int b = 0; b < cpw; b += 128) {
    const int cb = wave * cpw + 4 * kq + b;
    f32x4 hv[8], gv[8], sv[ADA ? 8 : 1], wv[8][NT];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      hv[u] = *(const f32x4 *)(hr + cb + 16 * u);
      gv[u] = *(const f32x4 *)(gr + cb + 16 * u);
      if constexpr (ADA) sv[u] = *(const f32x4 *)(sr + cb + 16 * u);
#pragma unroll
      for (int t = 0; t < NT; ++t) wv[u][t] = *(const f32x4 *)(wr[t] + cb + 16 * u);
    }
    __builtin_amdgcn_sched_barrier(0);  // keep the batch's loads ahead of its MFMAs
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        ss += hv[u][e] * hv[u][e];
        const float a = hv[u][e] * (ADA ? 1.0f + gv[u][e] : gv[u][e]);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, wv[u][t][e], acc[t], 0, 0, 0);
          if constexpr (ADA)
            acc2[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(sv[u][e], wv[u][t][e], acc2[t], 0, 0, 0);
        }
      }
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    part[wave][t][lane] = acc[t];
    if constexpr (ADA) part2[wave][t][lane] = acc2[t];
  }
  ssq[wave][lane] = ss;
  __syncthreads();
  // thread (i, j): token m0 + i, outputs 16 t + j; D[i][j] of a tile sits in
  // lane j + 16 (i / 4), component i % 4
  const int i = threadIdx.x >> 4, j = threadIdx.x & 15, m = m0 + i;
  if (m >= f.M) return;
  float s2 = 0.f;
#pragma unroll
  for (int w = 0; w < 4; ++w)
#pragma unroll
    for (int q = 0; q < 4; ++q) s2 += ssq[w][i + 16 * q];
  const float rstd = 1.0f / sqrtf(s2 / (float)f.d + f.eps);
  const int src = j + 16 * (i >> 2), cmp = i & 3;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int a = 16 * t + j;
    if (a < f.Da) {
      const float v = (part[0][t][src][cmp] + part[1][t][src][cmp]) + (part[2][t][src][cmp] + part[3][t][src][cmp]);
      float u = f.b_out[a];
      if constexpr (ADA)
        u += (part2[0][t][src][cmp] + part2[1][t][src][cmp]) + (part2[2][t][src][cmp] + part2[3][t][src][cmp]);
      euler_out(f, m, a, rstd * v + u);
    }
  }
}

// Distinct flow times of a batched step's tokens, by bits (one workgroup): a
// fleet's tokens share a handful of times, so the modulations (0.24 TFLOP and a
// 1.4 GB result per step at 3200 tokens of the 1024-wide expert) are computed
// once per time instead of once per token.  Keys go into an LDS hash table of
// four times kMaxTimeClasses slots; a token reads its slot before it tries the
// atomic, so equal times do not serialise.  More than kMaxTimeClasses distinct
// times: every token its own class.
constexpr int kMaxTimeClasses = 1024;
__global__ __launch_bounds__(1024) void time_classes_kernel(const float *__restrict__ t, int M,
                                                             int32_t *__restrict__ cls, float *__restrict__ cls_t,
                                                             int *__restrict__ n_cls) {
  constexpr unsigned SLOTS = 4 * kMaxTimeClasses, EMPTY = 0xFFFFFFFFu;
  __shared__ unsigned keys[SLOTS];
  __shared__ int ids[SLOTS];
  __shared__ int count;
  for (unsigned i = threadIdx.x; i < SLOTS; i += blockDim.x) keys[i] = EMPTY;
  if (threadIdx.x == 0) count = 0;
  __syncthreads();
  auto key_of = [&](int m) {
    const unsigned k = __float_as_uint(t[m]);
    return k == EMPTY ? 0x7FC00000u : k;  // that NaN as another
  };
  auto slot_of = [&](unsigned k) { return (k * 2654435761u) >> 20; };  // 12 bits
  static_assert(SLOTS == 4096, "slot_of");
  for (int m = threadIdx.x; m < M; m += blockDim.x) {
    const unsigned k = key_of(m);
    unsigned sl = slot_of(k);
    for (unsigned probe = 0; probe < SLOTS; ++probe, sl = (sl + 1) & (SLOTS - 1)) {
      unsigned cur = __hip_atomic_load(&keys[sl], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (cur == EMPTY) {
        if (__hip_atomic_load(&count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > kMaxTimeClasses) break;
        cur = atomicCAS(&keys[sl], EMPTY, k);
        if (cur == EMPTY) {
          ids[sl] = atomicAdd(&count, 1);
          break;
        }
      }
      if (cur == k) break;
    }
  }
  __syncthreads();
  const int n = count;
  if (n > kMaxTimeClasses) {
    for (int m = threadIdx.x; m < M; m += blockDim.x) {
      cls[m] = m;
      cls_t[m] = t[m];
    }
  } else {
    for (int m = threadIdx.x; m < M; m += blockDim.x) {
      const unsigned k = key_of(m);
      unsigned sl = slot_of(k);
      while (keys[sl] != k) sl = (sl + 1) & (SLOTS - 1);  // every key is in the table
      cls[m] = ids[sl];
    }
    for (unsigned i = threadIdx.x; i < SLOTS; i += blockDim.x)
      if (keys[i] != EMPTY) cls_t[ids[i]] = __uint_as_float(keys[i]);
  }
  if (threadIdx.x == 0) *n_cls = n > kMaxTimeClasses ? M : n;
}

// Sinusoidal time features of the distinct flow times (see time_feat_kernel).
__global__ __launch_bounds__(256) void class_feat_kernel(const float *__restrict__ cls_t, const int *__restrict__ n_cls,
                                                          int d, const float *__restrict__ freqs,
                                                          op_t *__restrict__ te, unsigned *status) {
  const int r = blockIdx.x, n = blockIdx.y * blockDim.x + threadIdx.x, half = d >> 1;
  if (r >= *n_cls || n >= half) return;
  const float arg = freqs[n] * cls_t[r];
  const int KB = d / kTileK;
  float sv, cv;
  sincosf(arg, &sv, &cv);
  unsigned bad = 0;
  store_op(te + afrag_index(r, n, KB), sv, bad);
  store_op(te + afrag_index(r, half + n, KB), cv, bad);
  flush_range(status, bad);
}

// Adaptive RMSNorm of a batched step as a pass of its own: the normalised
// operand RMS(h) (1 + a) + b in fp16, so that QKV and gate/up are one product of
// it instead of two (the scaled stream and the shift through the same weights).
// Bound by reading h: a workgroup takes 16 rows (whole fragment blocks), each
// thread 8 columns of one row at a time, h held in registers between the sum of
// squares and the output.  NI = 256-column passes (d <= 256 NI).
template <int NI>
__global__ __launch_bounds__(512) void ada_norm_kernel(const float *__restrict__ h, int M, int d, float eps,
                                                        const float *__restrict__ scale,
                                                        const float *__restrict__ shift, int mod_ld,
                                                        const int32_t *__restrict__ mod_row, op_t *__restrict__ next,
                                                        unsigned *status) {
  __shared__ float part[32][17];
  const int r = threadIdx.x & 15, cg = threadIdx.x >> 4;
  const int m = blockIdx.x * 16 + r, mc = min(m, M - 1);
  const size_t mr = (size_t)mod_row[mc] * mod_ld;
  f32x4 v[NI][2];
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int c = i * 256 + cg * 8;
    const bool ok = c < d;
    const float *p = h + (size_t)mc * d + (ok ? c : 0);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      v[i][q] = *(const f32x4 *)(p + 4 * q);
      if (ok) ss += v[i][q][0] * v[i][q][0] + v[i][q][1] * v[i][q][1] + v[i][q][2] * v[i][q][2] + v[i][q][3] * v[i][q][3];
    }
  }
  part[cg][r] = ss;
  __syncthreads();
  float s2 = 0.f;
#pragma unroll
  for (int q = 0; q < 32; ++q) s2 += part[q][r];
  const float rstd = 1.0f / sqrtf(s2 / (float)d + eps);
  unsigned bad = 0;
  const int KB = d / kTileK;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int c = i * 256 + cg * 8;
    if (c >= d || m >= M) continue;
    f16x8 o;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const f32x4 a = *(const f32x4 *)(scale + mr + c + 4 * q), b = *(const f32x4 *)(shift + mr + c + 4 * q);
      const f32x4 n = v[i][q] * rstd * (a + 1.0f) + b;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[4 * q + e] = (op_t)n[e];
      check_op4(n[0], n[1], n[2], n[3], bad);
    }
    *(f16x8 *)(next + afrag_index(m, c, KB)) = o;
  }
  flush_range(status, bad);
}

// Trajectory Reconciliation set-up: keep the initial noise x_0 and clear the
// velocity sums of the urgent tokens.
__global__ __launch_bounds__(256) void tr_init_kernel(TrArgs a) {
  const int n = a.B * a.H * a.Da;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    a.x0[i] = a.x[i];
    a.vsum[i] = 0.f;
  }
}

// Release after step K (Sec. 4.2): the urgent actions a^i = x_K^i, i < U, are
// copied out; with Trajectory Reconciliation (Sec. 4.3, Eq. 6) their internal
// states are then re-integrated under the canonical step,
// x'_K = x_0 + (1/N*) sum_k v_k, written in the flow-time convention of the
// integrator (dt* = -1/N*) and in the same form as its Euler update, so that
// with K = 1 the reconciled state equals the uniform schedule's x_1 bit for bit.
__global__ __launch_bounds__(256) void tr_release_kernel(TrArgs a) {
  const int n = a.B * a.U * a.Da;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const int c = i % a.Da;
    const int bu = i / a.Da;
    const int b = bu / a.U, u = bu - b * a.U;
    const size_t idx = ((size_t)b * a.H + u) * a.Da + c;
    const float v = a.x[idx];
    a.urgent[i] = v;
    if (a.urgent_host) a.urgent_host[i] = v;  // straight to the controller's pinned buffer
    if (a.reconcile) a.x[idx] = a.x0[idx] + a.dt_star * a.vsum[idx];
  }
  if (a.urgent_host) __threadfence_system();
}

// Ghost Action Correction (Sec. 4.4): E = sum_{i<U} (a'^i - a^i) over the ghost
// actions a'^i = x'^i_{N*} and released a^i (Eq. 8, summed in token order),
// then a^i = x^i_{N*} + E / (S - U) for i = U .. S-1 on the corrected
// dimensions (Eq. 9); executed[0..U) are the released actions unchanged.
__global__ __launch_bounds__(64) void gac_kernel(TrArgs a) {
  const int b = blockIdx.x;
  const int c = threadIdx.x;
  if (c >= a.Da) return;
  const float *xb = a.x + (size_t)b * a.H * a.Da;
  const float *ub = a.urgent + (size_t)b * a.U * a.Da;
  float *eb = a.executed + (size_t)b * a.S * a.Da;
  float E = 0.f;
  for (int i = 0; i < a.U; ++i) E += xb[(size_t)i * a.Da + c] - ub[(size_t)i * a.Da + c];
  const float shift = (a.gac_mask == nullptr || a.gac_mask[c] != 0) ? E / (float)(a.S - a.U) : 0.f;
  for (int i = 0; i < a.U; ++i) eb[(size_t)i * a.Da + c] = ub[(size_t)i * a.Da + c];
  for (int i = a.U; i < a.S; ++i) eb[(size_t)i * a.Da + c] = xb[(size_t)i * a.Da + c] + shift;
}

__global__ void stamp_kernel(uint64_t *dst) {
  if (threadIdx.x == 0) {
    const uint64_t now = __builtin_amdgcn_s_memrealtime();
    __hip_atomic_store(dst, now, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// fp32 to bf16, nearest-even; a NaN keeps its upper bits and turns quiet.
__device__ __forceinline__ uint16_t bf16_rne(uint32_t u) {
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)((u >> 16) | 0x40u);
  return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// 8 consecutive source elements from index i as bf16 bits.  VEC: the source is
// 16-byte aligned (i is a multiple of 8 then), else element loads.
template <bool F32, bool VEC>
__device__ __forceinline__ u16x8 load8_bf16(const void *src, size_t i) {
  u16x8 o;
  if constexpr (F32) {
    const uint32_t *p = (const uint32_t *)src + i;
    if constexpr (VEC) {
      const u32x4_t a = *(const u32x4_t *)p, b = *(const u32x4_t *)(p + 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        o[e] = bf16_rne(a[e]);
        o[4 + e] = bf16_rne(b[e]);
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = bf16_rne(p[e]);
    }
  } else {
    const uint16_t *p = (const uint16_t *)src + i;
    if constexpr (VEC) {
      o = *(const u16x8 *)p;
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = p[e];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e)  // signalling NaNs turn quiet, as from fp32
      if ((o[e] & 0x7FFFu) > 0x7F80u) o[e] |= 0x40u;
  }
  return o;
}

// Prefix K/V into the stores (see PrefixArgs): bound by memory, each value read
// and written once with 16-byte accesses.  It takes the place of a repacking
// on the host (device to host copy, scalar loops, copy back): a new prefix and
// its release together 11.10 -> 4.98 ms at batch 1 (18 layers, 816 keys, bf16)
// and 52.8 -> 2.38 ms at 16 environments (6 layers, fp32), same machine.  K rows are copied; the V block goes
// through LDS (rows padded by 16 bytes: the 64 lanes of a column read hit 64
// banks) and leaves as [hd][32 keys permuted], vt_key_pos: the 8 keys of 16-byte
// chunk g of a column are 4g..4g+3 and 16+4g..16+4g+3.
template <int HD, bool F32, bool VEC>
__global__ __launch_bounds__(256) void prefix_pack_kernel(PrefixArgs a) {
  __shared__ __align__(16) uint16_t vs[32][HD + 8];
  const int blk = a.blk0 + (int)(blockIdx.x % (unsigned)a.n_blk);
  const int eh = (int)(blockIdx.x / (unsigned)a.n_blk);
  const int b = eh / a.n_kv_heads, g = eh - b * a.n_kv_heads;
  const size_t dst_eh = (size_t)(a.env0 + b) * a.n_kv_heads + g;
  const size_t src = blockIdx.z * a.src_layer + b * a.src_env + (size_t)g * HD;
  __bf16 *kd = a.kc + blockIdx.z * a.dst_layer + (dst_eh * a.s_alloc + (size_t)blk * 32) * HD;
  __bf16 *vd = a.vtc + blockIdx.z * a.dst_layer + vt_index(dst_eh, blk * 32, 0, HD, a.s_alloc);
#pragma unroll
  for (int it = 0; it < HD / 64; ++it) {
    const int q = it * 256 + threadIdx.x;
    const int key = q / (HD / 8), c = (q % (HD / 8)) * 8;
    const int s = blk * 32 + key;
    u16x8 kv = {0, 0, 0, 0, 0, 0, 0, 0}, vv = kv;
    if (s < a.n_keys) {
      const size_t i = src + (size_t)(s - a.key0) * a.n_kv_heads * HD + c;
      kv = load8_bf16<F32, VEC>(a.k, i);
      vv = load8_bf16<F32, VEC>(a.v, i);
    }
    *(u16x8 *)(kd + key * HD + c) = kv;
    *(u16x8 *)&vs[key][c] = vv;
  }
  __syncthreads();
  for (int q = threadIdx.x; q < HD * 2; q += 256) {  // column pair q / 4, chunk q % 4
    const int c = (q >> 2) * 2, ch = q & 3;
    u16x8 o0, o1;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint32_t two = *(const uint32_t *)&vs[16 * (e >> 2) + 4 * ch + (e & 3)][c];
      o0[e] = (uint16_t)two;
      o1[e] = (uint16_t)(two >> 16);
    }
    *(u16x8 *)(vd + c * 32 + ch * 8) = o0;
    *(u16x8 *)(vd + (c + 1) * 32 + ch * 8) = o1;
  }
}

template <int HD>
static hipError_t launch_prefix_hd(const PrefixArgs &a, bool f32, hipStream_t s) {
  const dim3 grid((unsigned)(a.n_env * a.n_kv_heads * a.n_blk), 1, a.n_layers), wg(256);
  const bool vec = (((uintptr_t)a.k | (uintptr_t)a.v) & 15) == 0;  // rows are multiples of 128 bytes
  if (f32 && vec) hipLaunchKernelGGL((prefix_pack_kernel<HD, true, true>), grid, wg, 0, s, a);
  else if (f32) hipLaunchKernelGGL((prefix_pack_kernel<HD, true, false>), grid, wg, 0, s, a);
  else if (vec) hipLaunchKernelGGL((prefix_pack_kernel<HD, false, true>), grid, wg, 0, s, a);
  else hipLaunchKernelGGL((prefix_pack_kernel<HD, false, false>), grid, wg, 0, s, a);
  return hipGetLastError();
}

hipError_t launch_prefix_pack(const PrefixArgs &a, int head_dim, bool f32, hipStream_t s) {
  if (a.n_env < 1 || a.n_blk < 1 || a.n_layers < 1 || (a.blk0 + a.n_blk) * 32 > a.s_alloc) return hipErrorInvalidValue;
  const size_t esz = f32 ? 4 : 2;
  constexpr int kMaxZ = 32768;
  for (int l = 0; l < a.n_layers; l += kMaxZ) {
    const int r = for_pack_launches(a.n_env, a.n_kv_heads, a.n_blk, [&](int env, int envs, int blk, int blks) {
      PrefixArgs p = a;
      p.n_layers = a.n_layers - l < kMaxZ ? a.n_layers - l : kMaxZ;
      p.env0 = a.env0 + env; p.n_env = envs;
      p.blk0 = a.blk0 + blk; p.n_blk = blks;
      const size_t src = (l * a.src_layer + env * a.src_env) * esz;
      p.k = (const char *)a.k + src;
      p.v = (const char *)a.v + src;
      p.kc = a.kc + l * a.dst_layer;
      p.vtc = a.vtc + l * a.dst_layer;
      if (head_dim == 64) return (int)launch_prefix_hd<64>(p, f32, s);
      if (head_dim == 128) return (int)launch_prefix_hd<128>(p, f32, s);
      if (head_dim == 256) return (int)launch_prefix_hd<256>(p, f32, s);
      return (int)hipErrorInvalidValue;
    });
    if (r) return (hipError_t)r;
  }
  return hipSuccess;
}

hipError_t launch_temb(const float *x, const float *t, int M, int Da, int d, const float *w_in,
                       const float *b_in, const float *freqs, op_t *te, unsigned *status, hipStream_t s,
                       hipEvent_t ev0, hipEvent_t ev1, const int32_t *env_map, int chunk) {
  if (env_map && chunk < 1) return hipErrorInvalidValue;
  if (M >= 1024)
    UAD_LAUNCH(temb_kernel<16>, dim3((M + 15) / 16, (d + 255) / 256), dim3(256), 0, s, ev0, ev1, x, t, M, Da, d, w_in,
               b_in, freqs, te, status, env_map, chunk);
  else
    UAD_LAUNCH(temb_kernel<1>, dim3(M, (d + 255) / 256), dim3(256), 0, s, ev0, ev1, x, t, M, Da, d, w_in, b_in, freqs,
               te, status, env_map, chunk);
  return hipGetLastError();
}

hipError_t launch_temb_ada(const float *x, const float *t, int M, int Da, int d, const float *w_in,
                           const float *b_in, const float *freqs, op_t *te, float *h, float *ssq, int m_alloc,
                           unsigned *status, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1, const float *mod_a0,
                           int mod_ld, op_t *next) {
  if (mod_a0 && !next) return hipErrorInvalidValue;
  if (M >= 1024)
    UAD_LAUNCH(temb_ada_kernel<16>, dim3((M + 15) / 16, (d + 255) / 256), dim3(256), 0, s, ev0, ev1, x, t, M, Da, d,
               w_in, b_in, freqs, te, h, ssq, m_alloc, mod_a0, mod_ld, next, status);
  else
    UAD_LAUNCH(temb_ada_kernel<1>, dim3(M, (d + 255) / 256), dim3(256), 0, s, ev0, ev1, x, t, M, Da, d, w_in, b_in,
               freqs, te, h, ssq, m_alloc, mod_a0, mod_ld, next, status);
  return hipGetLastError();
}

// Time features of a whole schedule: row r = step * m_alloc + i takes the
// flow time t[step * M + i] (i < M), padding rows time 0.
__global__ __launch_bounds__(256) void time_feat_kernel(const float *__restrict__ t, int M, int m_alloc, int rows,
                                                         int d, const float *__restrict__ freqs,
                                                         op_t *__restrict__ te, unsigned *status) {
  const int r = blockIdx.x;
  const int n = blockIdx.y * blockDim.x + threadIdx.x;
  const int half = d >> 1;
  if (r >= rows || n >= half) return;
  const int st = r / m_alloc, i = r - st * m_alloc;
  const float tv = i < M ? t[(size_t)st * M + i] : 0.f;
  const float arg = freqs[n] * tv;
  const int KB = d / kTileK;
  float sv, cv;
  sincosf(arg, &sv, &cv);  // one range reduction for both
  unsigned bad = 0;
  store_op(te + afrag_index(r, n, KB), sv, bad);
  store_op(te + afrag_index(r, half + n, KB), cv, bad);
  flush_range(status, bad);
}

hipError_t launch_time_features(const float *t, int M, int m_alloc, int n_steps, int d, const float *freqs,
                                op_t *te, unsigned *status, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  if (M < 1 || m_alloc < M || m_alloc % 16 != 0 || n_steps < 1 || d % 64 != 0) return hipErrorInvalidValue;
  const int rows = n_steps * m_alloc;
  UAD_LAUNCH(time_feat_kernel, dim3(rows, (d / 2 + 255) / 256), dim3(256), 0, s, ev0, ev1, t, M, m_alloc, rows, d,
             freqs, te, status);
  return hipGetLastError();
}

hipError_t launch_time_classes(const float *t, int M, int32_t *cls, float *cls_t, int *n_cls, hipStream_t s,
                               hipEvent_t ev0, hipEvent_t ev1) {
  UAD_LAUNCH(time_classes_kernel, dim3(1), dim3(1024), 0, s, ev0, ev1, t, M, cls, cls_t, n_cls);
  return hipGetLastError();
}

hipError_t launch_class_features(const float *cls_t, const int *n_cls, int M, int d, const float *freqs, op_t *te,
                                 unsigned *status, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  UAD_LAUNCH(class_feat_kernel, dim3(M, (d / 2 + 255) / 256), dim3(256), 0, s, ev0, ev1, cls_t, n_cls, d, freqs, te,
             status);
  return hipGetLastError();
}

hipError_t launch_ada_norm(const float *h, int M, int d, float eps, const float *scale, const float *shift, int mod_ld,
                           const int32_t *mod_row, op_t *next, unsigned *status, hipStream_t s, hipEvent_t ev0,
                           hipEvent_t ev1) {
  if (d % 32 != 0) return hipErrorInvalidValue;
  const dim3 grid((M + 15) / 16), wg(512);
#define UAD_ADA_NORM(NI)                                                                                        \
  case NI:                                                                                                      \
    UAD_LAUNCH(ada_norm_kernel<NI>, grid, wg, 0, s, ev0, ev1, h, M, d, eps, scale, shift, mod_ld, mod_row, next, \
               status);                                                                                         \
    return hipGetLastError();
  switch ((d + 255) / 256) {
    UAD_ADA_NORM(1)
    UAD_ADA_NORM(2)
    UAD_ADA_NORM(3)
    UAD_ADA_NORM(4)
    UAD_ADA_NORM(5)
    UAD_ADA_NORM(6)
    UAD_ADA_NORM(7)
    UAD_ADA_NORM(8)
  }
#undef UAD_ADA_NORM
  return hipErrorInvalidValue;
}

hipError_t launch_final(const FinalArgs &f, bool mapped, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  if (mapped && (!f.mod_scale || !f.mod_row)) return hipErrorInvalidValue;
  if (f.M >= 1024 && !f.debug_field && f.d % 512 == 0 && f.Da <= 64) {
    const dim3 gr((f.M + 15) / 16);
    if (f.mod_scale && !mapped) return hipErrorInvalidValue;
    if (f.mod_scale) {
      switch ((f.Da + 15) / 16) {
        case 1: UAD_LAUNCH((final_mfma_kernel<1, true>), gr, dim3(256), 0, s, ev0, ev1, f); return hipGetLastError();
        case 2: UAD_LAUNCH((final_mfma_kernel<2, true>), gr, dim3(256), 0, s, ev0, ev1, f); return hipGetLastError();
        case 3: UAD_LAUNCH((final_mfma_kernel<3, true>), gr, dim3(256), 0, s, ev0, ev1, f); return hipGetLastError();
        case 4: UAD_LAUNCH((final_mfma_kernel<4, true>), gr, dim3(256), 0, s, ev0, ev1, f); return hipGetLastError();
      }
    }
    switch ((f.Da + 15) / 16) {
      case 1: UAD_LAUNCH((final_mfma_kernel<1, false>), gr, dim3(256), 0, s, ev0, ev1, f); return hipGetLastError();
      case 2: UAD_LAUNCH((final_mfma_kernel<2, false>), gr, dim3(256), 0, s, ev0, ev1, f); return hipGetLastError();
      case 3: UAD_LAUNCH((final_mfma_kernel<3, false>), gr, dim3(256), 0, s, ev0, ev1, f); return hipGetLastError();
      case 4: UAD_LAUNCH((final_mfma_kernel<4, false>), gr, dim3(256), 0, s, ev0, ev1, f); return hipGetLastError();
    }
  }
  const dim3 grid(f.M, (f.Da + kFinalOuts - 1) / kFinalOuts);
#define UAD_FINAL(NC)                                                                  \
  case NC:                                                                             \
    if (mapped)                                                                        \
      UAD_LAUNCH((final_kernel<NC, true>), grid, dim3(256), 0, s, ev0, ev1, f);        \
    else                                                                               \
      UAD_LAUNCH((final_kernel<NC, false>), grid, dim3(256), 0, s, ev0, ev1, f);       \
    break;
  switch ((f.d + 255) / 256) {
    UAD_FINAL(1)
    UAD_FINAL(2)
    UAD_FINAL(3)
    UAD_FINAL(4)
    UAD_FINAL(5)
    UAD_FINAL(6)
    UAD_FINAL(7)
    UAD_FINAL(8)
    default: return hipErrorInvalidValue;
  }
#undef UAD_FINAL
  return hipGetLastError();
}

hipError_t launch_tr_init(const TrArgs &a, hipStream_t s) {
  const int n = a.B * a.H * a.Da;
  hipLaunchKernelGGL(tr_init_kernel, dim3((n + 255) / 256), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_tr_release(const TrArgs &a, hipStream_t s) {
  const int n = a.B * a.U * a.Da;
  hipLaunchKernelGGL(tr_release_kernel, dim3((n + 255) / 256), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_gac(const TrArgs &a, hipStream_t s) {
  if (a.Da > 64) return hipErrorInvalidValue;
  hipLaunchKernelGGL(gac_kernel, dim3(a.B), dim3(64), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_stamp(uint64_t *dst, hipStream_t s) {
  hipLaunchKernelGGL(stamp_kernel, dim3(1), dim3(64), 0, s, dst);
  return hipGetLastError();
}

}  // namespace uad
