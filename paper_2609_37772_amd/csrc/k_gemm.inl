// Projection GEMMs of the action expert: C[M][N] = A[M][K] * W[N][K]^T on the
// gfx950 MFMA units (v_mfma_f32_16x16x32_f16), fp32 accumulation, with the
// epilogue of the layer fused in.
//
// Shape of the work: M is the token count (B*H: 16..3200), N and K are the
// projection sizes (256..8192).  At batch 1 a step streams ~0.6 GB of weights
// for ~50 tokens, and each CU's vector-memory pipe (not HBM) is what a
// workgroup waits on, so the work is cut to balance the bytes per workgroup:
//   * a workgroup owns T 16-column weight tiles over the full K and a group of
//     up to four 16-row tiles (batch 1: the ~50 rows are split over 2-3
//     workgroups, which re-read the weight tile from L2 instead of every
//     workgroup reading all rows of the activations);
//   * its waves cut K into runs of KPW 32-deep blocks and issue all loads of
//     a run (weights and activations) before its first MFMA;
//   * weights and activations are both stored in MFMA fragment order, so each
//     operand load is one aligned 16-byte load per lane, 1 KiB per wave;
//   * per-wave partial tiles are reduced through LDS in fixed wave order
//     (deterministic, no atomics).
// RMSNorm is folded into the GEMMs: the residual GEMMs (time-MLP out, O, down)
// update h for their columns, write every row's sum of squares over 16 columns (the
// batched kernels: over a wave's columns or an output tile) and the next operand
// fp16(h * gain_next); the GEMMs that consume a
// normalised input (QKV, gate/up) scale their accumulators by
// rstd[row] = (sum of those sums / d + eps)^-1/2, since
// RMSNorm(h) W^T = rstd * ((h * gain) W^T).
#include "uad_internal.h"

namespace uad {

// tanh-approximate GELU, 0.5 z (1 + tanh(u)) with u = sqrt(2/pi) (z + 0.044715 z^3),
// evaluated as z * sigmoid(2u) = z / (1 + 2^(-2u log2 e)) (the same function)
// with the hardware exp2 and reciprocal (~1 ulp each; the results are stored
// as fp16): an IEEE division here made the gate/up epilogue ALU-bound.  Large
// negative z gives -0 (2^t -> inf), large positive z gives z, NaN propagates.
__device__ __forceinline__ float gelu_tanh(float z) {
  const float k1 = -2.3022081983f;    // -2 sqrt(2/pi) log2(e)
  const float k2 = -0.1029432396f;    // k1 * 0.044715
  const float t = z * __builtin_fmaf(k2, z * z, k1);
  return z * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(t));
}

// SiLU z * sigmoid(z), by the same exp2 / reciprocal route
__device__ __forceinline__ float silu(float z) {
  return z * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950409f * z));
}

// Epilogue of one output element (row, col = 16 * tile + (ln & 15)) given its
// accumulated value v (and, for GeGLU, the matching up-projection value u);
// rs is the row's rstd (1 when unused).  EPI_RESID_F32 takes the residual h0,
// the next operand's scale sc and the branch gate gt, and must be called by
// the 16 lanes of a row together (sum of squares via shuffles).  BY_CLASS
// (EPI_MOD): modulations only, no operands of a step's norms.  (A test of the
// shift operands' pointer and their address from two 32-bit factors cost every
// element: 98.8 -> 101.6 us at 240 rows, 26624 columns, K = 1024.)
template <int EPI, bool BY_CLASS>
__device__ __forceinline__ void epilogue_elem(const GemmArgs &g, int row, bool row_ok, int tile, int ln, float v,
                                              float u, float rs, float h0, float sc, float gt, unsigned &bad) {
  if (EPI == EPI_MOD) {
    // column c: layer c / 6d, part (c % 6d) / d (0..5 = a, b, g of the
    // attention norm, then of the MLP norm), index c % d; the final norm's
    // (a, b) follow the layers
    const int col = tile * 16 + (ln & 15);
    if (row_ok) {
      const float mv = v + g.bias[col];
      ((float *)g.out)[(size_t)row * g.ldo + col] = mv;
      const int per_layer = 6 * g.d_model;
      const int l = col / per_layer;
      if (!BY_CLASS && l < g.n_layers) {
        const int r6 = col - l * per_layer;
        const int part = r6 / g.d_model, j = r6 - part * g.d_model;
        const int KBd = g.d_model / kTileK;
        if (part == 1 || part == 4)
          store_op(g.mod_shift_ops + (size_t)(2 * l + (part == 4)) * g.shift_stride + afrag_index(row, j, KBd), mv, bad);
        else if (part == 0 && l == 0 && g.next)
          store_op(g.next + afrag_index(row, j, KBd), g.h_in[(size_t)row * g.d_model + j] * (1.0f + mv), bad);
      }
    }
  } else if (EPI == EPI_RESID_F32) {
    const int col = tile * 16 + (ln & 15);
    float hv = 0.f;
    if (row_ok) {
      hv = (g.bias ? g.bias[col] : h0) + gt * v;
      ((float *)g.out)[(size_t)row * g.ldo + col] = hv;
    }
    float sq = hv * hv;  // sum over the 16 columns of this row (lanes sharing ln>>4)
    sq = sum_row16(sq);
    if (row_ok) {
      if ((ln & 15) == 0) g.ssq[(size_t)tile * g.m_alloc + row] = sq;
      if (g.mod_scale_next || g.gain_next) store_op(g.next + afrag_index(row, col, g.N / kTileK), hv * sc, bad);
    }
  } else if (row_ok) {
    if (EPI == EPI_GEGLU) {
      const int col = (tile >> 1) * 16 + (ln & 15);
      store_op((op_t *)g.out + afrag_index(row, col, g.ldo / kTileK), gelu_tanh(v * rs) * (u * rs), bad);
    } else {
      const int col = tile * 16 + (ln & 15);
      if (EPI == EPI_BIAS_SILU) {
        store_op((op_t *)g.out + afrag_index(row, col, g.ldo / kTileK), silu(v + g.bias[col]), bad);
      } else if (EPI == EPI_QKV) {
        v *= rs;
        if (col < g.q_dim) {
          ((__bf16 *)g.out)[(size_t)row * g.ldo + col] = (__bf16)v;
        } else {
          const int b = row / g.chunk, i = row - b * g.chunk;
          const int bp = g.env_map ? g.env_map[b] : b;  // the environment's K/V store slot
          const int kvd = g.n_kv_heads * g.head_dim;
          const int c2 = col - g.q_dim;
          const bool is_v = c2 >= kvd;
          const int c3 = is_v ? c2 - kvd : c2;
          const int kvh = c3 / g.head_dim, c = c3 - kvh * g.head_dim;
          const size_t env_head = (size_t)bp * g.n_kv_heads + kvh;
          const int s = g.prefix + i;
          if (!is_v)
            g.kc[(env_head * g.s_alloc + s) * g.head_dim + c] = (__bf16)v;
          else
            g.vtc[vt_index(env_head, s, c, g.head_dim, g.s_alloc)] = (__bf16)v;
        }
      }
    }
  }
}

constexpr int kMaxTilesPerGroup = 4;
constexpr int kMaxSsqTiles = 2048 / 16;  // d_model <= 2048

static int g_n_cu = 256;  // compute units of the device (set by gemm_init)

// PIPE (more than one pass, single operand): the operand registers are
// double buffered, so the loads of pass p + 1 are in flight while the MFMAs
// of pass p run and a launch pays one memory round trip instead of one per
// pass.
// MAP: g.mod_row / g.m_dev are in use (batched adaptive norm; an instance of its
// own, since the test alone cost the batch-1 residual projections 0.5 us each).
template <int EPI, int T, int KPW, bool DUAL, bool PIPE, bool MAP>
__global__ __launch_bounds__(512) void gemm_kernel(GemmArgs g) {
  static_assert(!(PIPE && DUAL), "double-buffered passes: single operand only");
  extern __shared__ float red[];  // [waves][4*T*4 slots][64 lanes]
  constexpr bool kRstd = (EPI == EPI_QKV || EPI == EPI_GEGLU);
  __shared__ float ssq_s[kRstd ? kMaxSsqTiles : 1][64];  // this group's rows' per-tile sums of squares
  __shared__ float rstd_s[64];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int waves = blockDim.x >> 6;
  const int tile0 = blockIdx.x * T;  // first 16-column weight tile
  const int MT = (g.M + 15) >> 4;
  const int mt0 = (blockIdx.z * MT) / gridDim.z;
  const int nmt = ((blockIdx.z + 1) * MT) / gridDim.z - mt0;  // 1..4, uniform
  const int m0 = mt0 * 16;
  const int KB = g.K / kTileK;
  const int passes = KB / (KPW * waves);
  if constexpr (MAP && EPI != EPI_RESID_F32) {
    g.M = min(g.M, *g.m_dev);
    if (m0 >= g.M) return;  // whole workgroup
  }

  f32x4 acc[kMaxTilesPerGroup][T], acc2[kMaxTilesPerGroup][DUAL ? T : 1];
#pragma unroll
  for (int mt = 0; mt < kMaxTilesPerGroup; ++mt) {
#pragma unroll
    for (int t = 0; t < T; ++t) acc[mt][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < (DUAL ? T : 1); ++t) acc2[mt][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // Operand loads of one pass (a run of KPW k-blocks per wave) and its MFMAs.
  f16x8 w[KPW][T], a[KPW][kMaxTilesPerGroup], a2[KPW][DUAL ? kMaxTilesPerGroup : 1];
  f16x8 wb[PIPE ? KPW : 1][T], ab[PIPE ? KPW : 1][kMaxTilesPerGroup];  // PIPE: the second buffer
  auto load_into = [&](int pass, auto &w, auto &a) {
    const int kb0 = (pass * waves + wave) * KPW;
    const op_t *wp = g.W + ((size_t)tile0 * KB + kb0) * kBlockElems + lane * 8;
#pragma unroll
    for (int j = 0; j < KPW; ++j)
#pragma unroll
      for (int t = 0; t < T; ++t) w[j][t] = *(const f16x8 *)(wp + ((size_t)t * KB + j) * kBlockElems);
    const op_t *ap = g.A + ((size_t)mt0 * KB + kb0) * kBlockElems + lane * 8;
#pragma unroll
    for (int mt = 0; mt < kMaxTilesPerGroup; ++mt) {
      if (mt >= nmt) break;  // wave-uniform: no instructions for the group's absent row tiles
      const bool ok = (m0 + mt * 16 + (lane & 15)) < g.M;
#pragma unroll
      for (int j = 0; j < KPW; ++j) a[j][mt] = ok ? *(const f16x8 *)(ap + ((size_t)mt * KB + j) * kBlockElems) : f16x8{};
      if constexpr (DUAL) {
        const op_t *ap2 = g.A2 + ((size_t)mt0 * KB + kb0) * kBlockElems + lane * 8;
#pragma unroll
        for (int j = 0; j < KPW; ++j)
          a2[j][mt] = ok ? *(const f16x8 *)(ap2 + ((size_t)mt * KB + j) * kBlockElems) : f16x8{};
      }
    }
  };
  auto mma_from = [&](const auto &w, const auto &a) {
#pragma unroll
    for (int mt = 0; mt < kMaxTilesPerGroup; ++mt) {
      if (mt >= nmt) break;
#pragma unroll
      for (int j = 0; j < KPW; ++j)
#pragma unroll
        for (int t = 0; t < T; ++t) {
          acc[mt][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[j][mt], w[j][t], acc[mt][t], 0, 0, 0);
          if (DUAL)
            acc2[mt][DUAL ? t : 0] =
                __builtin_amdgcn_mfma_f32_16x16x32_f16(a2[j][mt], w[j][t], acc2[mt][DUAL ? t : 0], 0, 0, 0);
        }
    }
  };

  // The first pass's operand loads go out first: any wait for the loads
  // issued after them (norm statistics, epilogue operands) covers them too,
  // so the kernel pays one memory round trip before its first MFMA.
  load_into(0, w, a);
  // Every global load the kernel needs is issued before the first use so a
  // launch costs one memory round trip:
  //  * rstd of this group's rows comes from the residual GEMM's per-tile sums
  //    of squares; they go straight to LDS (LDS-direct loads, 64 rows of one
  //    tile per wave instruction), so they hold no registers and nothing waits
  //    on them before the main loop is done;
  //  * the residual epilogue's h, gain / modulation and gate values of this
  //    thread's first kEpiPrefetch output elements.
  if (kRstd && g.use_rstd) {
    const int srow = min(m0 + lane, g.M - 1);
    for (int j = wave; j < g.ssq_tiles; j += waves)
      __builtin_amdgcn_global_load_lds((const void *)(g.ssq + (size_t)j * g.m_alloc + srow),
                                       (__attribute__((address_space(3))) void *)&ssq_s[j][0], 4, 0, 0);
  }
  const int n_out_all = (EPI == EPI_GEGLU) ? nmt * 256 * (T / 2) : nmt * 256 * T;
  constexpr int kEpiPrefetch = 2;
  float pre_h[kEpiPrefetch], pre_s[kEpiPrefetch], pre_g[kEpiPrefetch];
  if (EPI == EPI_RESID_F32) {
    // branch-free: every load is unconditional from a valid address (h itself
    // stands in for an absent operand) and the value is selected afterwards
    const bool has_mod = g.mod_scale_next != nullptr, has_gain = g.gain_next != nullptr;
    const bool has_gate = g.mod_gate != nullptr;
#pragma unroll
    for (int it = 0; it < kEpiPrefetch; ++it) {
      const int e = it * (int)blockDim.x + threadIdx.x;
      const int ln = e & 63, slot = e >> 6;
      const int r = slot & 3, t = (slot >> 2) % T, mt = min((slot >> 2) / T, kMaxTilesPerGroup - 1);
      const int row = min(m0 + mt * 16 + (ln >> 4) * 4 + r, g.M - 1);
      const int col = min((tile0 + t) * 16 + (ln & 15), g.N - 1);
      const float *hp = (const float *)g.out + (size_t)row * g.ldo + col;
      const size_t ro = (size_t)(MAP ? g.mod_row[row] : row) * g.mod_ld + col;
      const float *sp = has_mod ? g.mod_scale_next + ro : (has_gain ? g.gain_next + col : hp);
      const float *gp = has_gate ? g.mod_gate + ro : hp;
      const float hv = *hp, sv = *sp, gv = *gp;
      pre_h[it] = hv;
      pre_s[it] = has_mod ? 1.0f + sv : (has_gain ? sv : 0.f);
      pre_g[it] = has_gate ? gv : 1.0f;
    }
  }

  if constexpr (PIPE) {
    for (int pass = 0; pass < passes; pass += 2) {
      if (pass + 1 < passes) load_into(pass + 1, wb, ab);
      mma_from(w, a);
      if (pass + 1 < passes) {
        if (pass + 2 < passes) load_into(pass + 2, w, a);
        mma_from(wb, ab);
      }
    }
  } else {
    for (int pass = 0; pass < passes; ++pass) {
      if (pass > 0) load_into(pass, w, a);
      mma_from(w, a);
    }
  }

  if (kRstd && g.use_rstd) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the LDS-direct sums landed

  // Dual operand (normalised input = rstd * A + A2): fold rstd into each
  // wave's partial tile before the cross-wave reduction (it is linear).
  if (DUAL) {
    __syncthreads();  // ssq_s complete
    if (threadIdx.x < 64) {
      float ss = 0.f;
      for (int j = 0; j < g.ssq_tiles; ++j) ss += ssq_s[j][threadIdx.x];
      rstd_s[threadIdx.x] = 1.0f / sqrtf(ss / (float)g.K + g.eps);
    }
    __syncthreads();
#pragma unroll
    for (int mt = 0; mt < kMaxTilesPerGroup; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float rs = rstd_s[mt * 16 + (lane >> 4) * 4 + r];
#pragma unroll
        for (int t = 0; t < T; ++t) acc[mt][t][r] = rs * acc[mt][t][r] + acc2[mt][DUAL ? t : 0][r];
      }
  }

  // Cross-wave reduction through LDS, fixed order over waves.
  constexpr int SLOTS = kMaxTilesPerGroup * T * 4;  // (mt, t, r) triples per lane
#pragma unroll
  for (int mt = 0; mt < kMaxTilesPerGroup; ++mt) {
    if (mt >= nmt) break;  // the epilogue reads only the group's own row tiles
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[((wave * SLOTS) + (mt * T + t) * 4 + r) * 64 + lane] = acc[mt][t][r];
  }
  __syncthreads();
  if (!DUAL && kRstd && g.use_rstd && threadIdx.x < 64) {
    float ss = 0.f;
    for (int j = 0; j < g.ssq_tiles; ++j) ss += ssq_s[j][threadIdx.x];
    rstd_s[threadIdx.x] = 1.0f / sqrtf(ss / (float)g.K + g.eps);
  }
  __syncthreads();

  // Epilogue. Element e = slot*64 + lane with slot = (mt*T + t)*4 + r (for
  // GeGLU slot = (mt*(T/2) + pair)*4 + r); the D fragment of a 16x16 MFMA holds
  // row 4*(lane>>4)+r, column lane&15.  The per-wave trip count is uniform and
  // the 16 lanes holding one row are always active together.
  const int n_out = n_out_all;
  unsigned bad = 0;  // fp16 range flag of this thread's stores
  for (int e0 = 0, it = 0; e0 < n_out; e0 += blockDim.x, ++it) {
    const int e = e0 + threadIdx.x;
    if (e >= n_out) continue;  // whole waves only (n_out and blockDim are multiples of 64)
    const int ln = e & 63;
    const int slot = e >> 6;
    int mt, t, r;
    if (EPI == EPI_GEGLU) {
      r = slot & 3;
      const int q = slot >> 2;
      t = 2 * (q % (T / 2));
      mt = q / (T / 2);
    } else {
      r = slot & 3;
      t = (slot >> 2) % T;
      mt = (slot >> 2) / T;
    }
    const int rl = mt * 16 + (ln >> 4) * 4 + r;  // row within the group
    const int row = m0 + rl;
    const bool row_ok = row < g.M;
    const int s0 = (mt * T + t) * 4 + r;
    float v = 0.f;
    for (int w2 = 0; w2 < waves; ++w2) v += red[(w2 * SLOTS + s0) * 64 + ln];
    float u = 0.f, h0 = 0.f, sc = 0.f, gt = 1.f;
    if (EPI == EPI_GEGLU) {
      const int s1 = (mt * T + t + 1) * 4 + r;
      for (int w2 = 0; w2 < waves; ++w2) u += red[(w2 * SLOTS + s1) * 64 + ln];
    }
    if (EPI == EPI_RESID_F32) {
#pragma unroll
      for (int k = 0; k < kEpiPrefetch; ++k)
        if (it == k) { h0 = pre_h[k]; sc = pre_s[k]; gt = pre_g[k]; }
      if (it >= kEpiPrefetch && row_ok) {
        const int col = (tile0 + t) * 16 + (ln & 15);
        const size_t ro = (size_t)(MAP ? g.mod_row[row] : row) * g.mod_ld + col;
        h0 = g.bias ? 0.f : ((const float *)g.out)[(size_t)row * g.ldo + col];
        sc = g.mod_scale_next ? 1.0f + g.mod_scale_next[ro] : (g.gain_next ? g.gain_next[col] : 0.f);
        gt = g.mod_gate ? g.mod_gate[ro] : 1.0f;
      }
    }
    const float rs = (!DUAL && kRstd && g.use_rstd && row_ok) ? rstd_s[rl] : 1.0f;
    epilogue_elem<EPI, MAP && EPI == EPI_MOD>(g, row, row_ok, tile0 + t, ln, v, u, rs, h0, sc, gt, bad);
  }
  flush_range(g.status, bad);
}

template <int EPI, int T, int KPW>
static hipError_t launch_t(const GemmArgs &g, const GemmPlan &p, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  dim3 grid(g.N / kTileN / T, 1, p.mgroups);
  const uint32_t lds = (uint32_t)(p.waves * kMaxTilesPerGroup * T * 4 * 64 * sizeof(float));
  if constexpr (EPI == EPI_QKV || EPI == EPI_GEGLU) {
    if (g.A2) {
      if (!g.use_rstd) return hipErrorInvalidValue;
      UAD_LAUNCH((gemm_kernel<EPI, T, KPW, true, false, false>), grid, dim3(p.waves * 64), lds, s, ev0, ev1, g);
      return hipGetLastError();
    }
  }
  if constexpr (EPI == EPI_RESID_F32 || EPI == EPI_BIAS_SILU || EPI == EPI_MOD) {
    if (EPI == EPI_RESID_F32 ? g.mod_row != nullptr : g.m_dev != nullptr) {
      UAD_LAUNCH((gemm_kernel<EPI, T, KPW, false, false, true>), grid, dim3(p.waves * 64), lds, s, ev0, ev1, g);
      return hipGetLastError();
    }
  }
  // Double-buffered passes hold ~200 registers, one 8-wave workgroup per CU:
  // only when the grid has no more workgroups than CUs (batch 1: down 4
  // passes, O 2; step 0.700 -> 0.696 ms same-machine; at 8 environments, 448
  // workgroups, they lost 4% against two co-resident workgroups per CU).
  if (p.passes > 1 && (long)grid.x * grid.z <= g_n_cu)
    UAD_LAUNCH((gemm_kernel<EPI, T, KPW, false, true, false>), grid, dim3(p.waves * 64), lds, s, ev0, ev1, g);
  else
    UAD_LAUNCH((gemm_kernel<EPI, T, KPW, false, false, false>), grid, dim3(p.waves * 64), lds, s, ev0, ev1, g);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Register-streamed kernel (time MLP in, modulations, and the residual
// projections that no ring shape takes): a workgroup owns a 128-row x
// 16*CT-column output tile over the full K; its 4 waves (2 x 2) each own
// 64 rows x 8*CT columns (4 x CT/2 MFMA 16x16x32 tiles).  No LDS for the
// operands: every wave streams its own fragment-order 1 KiB blocks straight
// into registers, kBigPD k-blocks ahead of the MFMAs (one aligned 16-byte
// load per lane and block; the two waves sharing a row or column panel find
// it in L2).  On 2048..3200-row projections this runs at 590-940 TFLOP/s without
// epilogue, against ~150 for the same tiles staged through a double-buffered
// LDS ring: there every 32-deep k-step waited out a full memory round trip,
// and __syncthreads' release fence drains all loads in flight, so deeper
// rings need a raw barrier.  Tiles are dealt to the 8 XCDs in contiguous
// runs, column-major over groups of 8 row panels, so the workgroups sharing
// an L2 share weight and activation panels.  The epilogue runs from the
// accumulators (no cross-wave reduction).
// ---------------------------------------------------------------------------
constexpr int kBigRowTiles = 8;  // 128 rows per workgroup
constexpr int kBigPD = 3;        // k-blocks in flight per wave

// Output tile of workgroup blockIdx.x over ceil(M / rows) row panels and tn
// column panels: XCD x = blockIdx % 8 takes a contiguous run of tiles,
// column-major over groups of 8 row panels, so the workgroups sharing an L2
// share weight and activation panels.  The grid has 8 * ceil(tiles / 8)
// workgroups (grid_tile_wgs); false for the padding ones.
__host__ __device__ __forceinline__ int grid_tile_wgs(int M, int rows, int tn) {
  return ((M + rows - 1) / rows * tn + 7) / 8 * 8;
}

__device__ __forceinline__ bool grid_tile_at(int wg, int M, int rows, int tn, int &pm, int &pn) {
  const int tm = (M + rows - 1) / rows, T = tm * tn;
  const int per = (T + 7) / 8;
  const int t = (wg & 7) * per + (wg >> 3);
  if (t >= T) return false;
  constexpr int GM = 8;
  const int grp = t / (GM * tn), in = t - grp * GM * tn;
  const int gm0 = grp * GM, gms = min(GM, tm - gm0);
  pm = gm0 + in % gms;
  pn = in / gms;
  return true;
}

__device__ __forceinline__ bool grid_tile(int M, int rows, int tn, int &pm, int &pn) {
  return grid_tile_at((int)blockIdx.x, M, rows, tn, pm, pn);
}

template <int CT>
__device__ __forceinline__ bool big_tile(const GemmArgs &g, int &mt0, int &nt0) {
  int pm, pn;
  if (!grid_tile(g.M, 16 * kBigRowTiles, g.N / (16 * CT), pm, pn)) return false;
  mt0 = pm * kBigRowTiles;
  nt0 = pn * CT;
  return true;
}

// Epilogue of the batched kernel.  The MFMA runs with the operands swapped
// (it accumulates C^T tiles), so lane l of tile (i, j) holds row l & 15 and
// the 4 consecutive columns 4 * (l >> 4) + 0..3: every fp32 access is one
// 16-byte load or store and every fp16 / bf16 store 8 bytes.  mt / nt are
// the wave's first row / column tile; rstd (when not null) the rstd of its
// TA*16 rows.
__device__ __forceinline__ f32x4 ld4(const float *p) { return *(const f32x4 *)p; }
__device__ __forceinline__ void st4(float *p, f32x4 v) { *(f32x4 *)p = v; }
__device__ __forceinline__ void st4h(op_t *p, f32x4 v, unsigned &bad) {
  *(f16x4 *)p = f16x4{(op_t)v[0], (op_t)v[1], (op_t)v[2], (op_t)v[3]};
  check_op4(v[0], v[1], v[2], v[3], bad);
}

// Residual epilogue, store half, over NI row tiles starting at i0: h = h0 (or
// bias) + gate * v, each row's sum of squares of h over the wave's columns (to
// ssq[row - ssq_row0]), next operand
// fp16(h * scale), scale = gain_next (one row [TB]).  ADA: the gate is a
// per-token modulation and the next norm a pass of its own (no next operand);
// else gate = 1.
template <int NI, bool ADA, int TA, int TB>
__device__ __forceinline__ void big_resid_store(const GemmArgs &g, const f32x4 (&acc)[TA][TB], int i0, int mt, int nt,
                                                int lane, const f32x4 (&h0)[NI][TB],
                                                const f32x4 (&gt)[ADA ? NI : 1][TB],
                                                const f32x4 (&sc)[TB], float *ssq, int ssq_row0, unsigned &bad) {
  float *h = (float *)g.out;
  const bool has_next = !ADA && g.gain_next != nullptr;
  const int csub = 4 * (lane >> 4);
  const int KBn = g.N / kTileK;
#pragma unroll
  for (int ii = 0; ii < NI; ++ii) {
    const int row = (mt + i0 + ii) * 16 + (lane & 15);
    const bool row_ok = row < g.M;
    float sq = 0.f;
#pragma unroll
    for (int j = 0; j < TB; ++j) {
      const int col = (nt + j) * 16 + csub;
      const f32x4 hv = ADA ? h0[ii][j] + gt[ADA ? ii : 0][j] * acc[i0 + ii][j] : h0[ii][j] + acc[i0 + ii][j];
      if (row_ok) st4(h + (size_t)row * g.ldo + col, hv);
      sq += hv[0] * hv[0] + hv[1] * hv[1] + hv[2] * hv[2] + hv[3] * hv[3];
      if (row_ok && has_next) st4h(g.next + afrag_index(row, col, KBn), hv * sc[j], bad);
    }
    // this wave's columns of the row: the 4 lanes holding them
    sq = sum_pair32(sum_pair16(sq));
    if (row_ok && lane < 16) ssq[row - ssq_row0] = sq;
  }
}

// Residual epilogue, load half: h0 (or the bias) of NI row tiles from i0, and
// the next operand's scale or (ADA) the gate.  Branch-free: every load
// comes from a valid address (an absent operand is stood in for by one that
// exists) and the value is selected afterwards, so no load waits on another.
template <int NI, bool ADA, int TB>
__device__ __forceinline__ void big_resid_load(const GemmArgs &g, int i0, int mt, int nt, int lane,
                                               f32x4 (&h0)[NI][TB], f32x4 (&gt)[ADA ? NI : 1][TB], f32x4 (&sc)[TB]) {
  const int csub = 4 * (lane >> 4);
  const bool has_next = g.gain_next != nullptr;
  const float *hb = g.bias ? g.bias : (const float *)g.out;
  const size_t hld = g.bias ? 0 : (size_t)g.ldo;
  const float *sb = has_next ? g.gain_next : hb;
  size_t mr[ADA ? NI : 1];  // the rows' modulation rows, loaded ahead of what they address
  if constexpr (ADA)
#pragma unroll
    for (int ii = 0; ii < NI; ++ii)
      mr[ii] = (size_t)g.mod_row[min((mt + i0 + ii) * 16 + (lane & 15), g.M - 1)] * g.mod_ld;
#pragma unroll
  for (int ii = 0; ii < NI; ++ii) {
    const int rowc = min((mt + i0 + ii) * 16 + (lane & 15), g.M - 1);
#pragma unroll
    for (int j = 0; j < TB; ++j) {
      const int col = (nt + j) * 16 + csub;
      h0[ii][j] = ld4(hb + (size_t)rowc * hld + col);
      if constexpr (ADA) {
        gt[ii][j] = ld4(g.mod_gate + mr[ii] + col);
      } else if (ii == 0) {
        const f32x4 sv = ld4(sb + col);
        sc[j] = has_next ? sv : f32x4{0.f, 0.f, 0.f, 0.f};
      }
    }
  }
}

// Residual epilogue over NI row tiles starting at i0, loads then stores.  All
// loads of the block are issued before its first store (the h stores may alias
// h0 loads of other rows, so the compiler would not hoist them).
template <int NI, bool ADA, int TA, int TB>
__device__ __forceinline__ void big_resid_rows(const GemmArgs &g, f32x4 (&acc)[TA][TB], int i0, int mt, int nt,
                                               int lane, float *ssq, int ssq_row0, unsigned &bad) {
  f32x4 h0[NI][TB], gt[ADA ? NI : 1][TB], sc[TB];
  big_resid_load<NI, ADA, TB>(g, i0, mt, nt, lane, h0, gt, sc);
  big_resid_store<NI, ADA, TA, TB>(g, acc, i0, mt, nt, lane, h0, gt, sc, ssq, ssq_row0, bad);
}

template <int EPI, int TA, int TB, int I0 = 0, int NI = TA>
__device__ __forceinline__ void big_epilogue(const GemmArgs &g, f32x4 (&acc)[TA][TB], int mt, int nt, int lane,
                                             const float *rstd, unsigned &bad, float *ssq_lds = nullptr,
                                             int ssq_row0 = 0) {
  const int csub = 4 * (lane >> 4);
  if constexpr (EPI == EPI_RESID_F32) {
    float *ssq = ssq_lds ? ssq_lds : g.ssq + (size_t)(nt / TB) * g.m_alloc;
    if (g.mod_gate) {
      constexpr int HB = NI % 2 == 0 ? 2 : 1;
#pragma unroll
      for (int i = I0; i < I0 + NI; i += HB) big_resid_rows<HB, true>(g, acc, i, mt, nt, lane, ssq, ssq_row0, bad);
    } else {
      // the whole tile in two halves: all of its h0 at once would cost the
      // main loop its second wave per SIMD (a half tile goes in one piece)
      constexpr int HB = NI == TA ? TA / 2 : NI;
#pragma unroll
      for (int i = I0; i < I0 + NI; i += HB) big_resid_rows<HB, false>(g, acc, i, mt, nt, lane, ssq, ssq_row0, bad);
    }
  } else if constexpr (EPI == EPI_QKV) {
    const int kvd = g.n_kv_heads * g.head_dim;
#pragma unroll
    for (int i = I0; i < I0 + NI; ++i) {
      const int row = (mt + i) * 16 + (lane & 15);
      if (row >= g.M) continue;
      const float rs = rstd ? rstd[i * 16 + (lane & 15)] : 1.0f;
      const int b = row / g.chunk, s = g.prefix + (row - b * g.chunk);
      const int bp = g.env_map ? g.env_map[b] : b;  // the environment's K/V store slot
#pragma unroll
      for (int j = 0; j < TB; ++j) {
        const int col = (nt + j) * 16 + csub;
        const f32x4 v = acc[i][j] * rs;
        if ((nt + j) * 16 < g.q_dim) {
          *(bf16x4 *)((__bf16 *)g.out + (size_t)row * g.ldo + col) =
              bf16x4{(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
        } else {
          const int c2 = col - g.q_dim;
          const bool is_v = c2 >= kvd;
          const int c3 = is_v ? c2 - kvd : c2;
          const int kvh = c3 / g.head_dim, c = c3 - kvh * g.head_dim;
          const size_t eh = (size_t)bp * g.n_kv_heads + kvh;
          if (!is_v) {
            *(bf16x4 *)(g.kc + (eh * g.s_alloc + s) * g.head_dim + c) =
                bf16x4{(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) g.vtc[vt_index(eh, s, c + r, g.head_dim, g.s_alloc)] = (__bf16)v[r];
          }
        }
      }
    }
  } else if constexpr (EPI == EPI_GEGLU) {
    const int KBo = g.ldo / kTileK;
#pragma unroll
    for (int i = I0; i < I0 + NI; ++i) {
      const int row = (mt + i) * 16 + (lane & 15);
      if (row >= g.M) continue;
      const float rs = rstd ? rstd[i * 16 + (lane & 15)] : 1.0f;
#pragma unroll
      for (int j = 0; j < TB; j += 2) {  // gate tile j, its up tile j + 1
        const int col = ((nt + j) >> 1) * 16 + csub;
        const f32x4 a = acc[i][j] * rs, u = acc[i][j + 1] * rs;
        st4h((op_t *)g.out + afrag_index(row, col, KBo),
             f32x4{gelu_tanh(a[0]) * u[0], gelu_tanh(a[1]) * u[1], gelu_tanh(a[2]) * u[2], gelu_tanh(a[3]) * u[3]},
             bad);
      }
    }
  } else if constexpr (EPI == EPI_BIAS_SILU) {
    const int KBo = g.ldo / kTileK;
    f32x4 bias[TB];
#pragma unroll
    for (int j = 0; j < TB; ++j) bias[j] = ld4(g.bias + (nt + j) * 16 + csub);
#pragma unroll
    for (int i = I0; i < I0 + NI; ++i) {
      const int row = (mt + i) * 16 + (lane & 15);
      if (row >= g.M) continue;
#pragma unroll
      for (int j = 0; j < TB; ++j) {
        const f32x4 z = acc[i][j] + bias[j];
        st4h((op_t *)g.out + afrag_index(row, (nt + j) * 16 + csub, KBo),
             f32x4{silu(z[0]), silu(z[1]), silu(z[2]), silu(z[3])}, bad);
      }
    }
  } else if constexpr (EPI == EPI_MOD) {
    // column c: layer c / 6d, part (c % 6d) / d (a, b, g of the attention
    // norm, then of the MLP norm), index c % d; a 16-column tile lies in one
    // part; the final norm's (a, b) follow the layers
    const int per_layer = 6 * g.d_model, KBd = g.d_model / kTileK;
    f32x4 bias[TB];
#pragma unroll
    for (int j = 0; j < TB; ++j) bias[j] = ld4(g.bias + (nt + j) * 16 + csub);
#pragma unroll
    for (int i = I0; i < I0 + NI; ++i) {
      const int row = (mt + i) * 16 + (lane & 15);
      if (row >= g.M) continue;
#pragma unroll
      for (int j = 0; j < TB; ++j) {
        const int col = (nt + j) * 16 + csub;
        const f32x4 mv = acc[i][j] + bias[j];
        st4((float *)g.out + (size_t)row * g.ldo + col, mv);
        const int l = col / per_layer;
        if (l < g.n_layers) {
          const int r6 = col - l * per_layer;
          const int part = r6 / g.d_model, jc = r6 - part * g.d_model;
          if (g.mod_shift_ops && (part == 1 || part == 4))
            st4h(g.mod_shift_ops + (size_t)(2 * l + (part == 4)) * g.shift_stride + afrag_index(row, jc, KBd), mv, bad);
          else if (part == 0 && l == 0 && g.next)
            st4h(g.next + afrag_index(row, jc, KBd), ld4(g.h_in + (size_t)row * g.d_model + jc) * (mv + 1.0f), bad);
        }
      }
    }
  }
}

// KS = 2 (when the output tiles fill at most one round of CUs, so that a
// 4-wave workgroup would leave each SIMD a single wave): 8 waves, waves
// 4..7 take the odd k-blocks of the same tile; the two partial tiles are
// summed through LDS and each k-half then runs the epilogue of half the
// wave's row tiles.
template <int EPI, int CT, int KS = 1>
__global__ __launch_bounds__(256 * KS) void gemm_big_kernel(GemmArgs g) {
  constexpr int TA = kBigRowTiles / 2, TB = CT / 2, PD = kBigPD;
  static_assert(EPI == EPI_BIAS_SILU || EPI == EPI_RESID_F32 || EPI == EPI_MOD, "QKV and gate/up run on the ring");
  static_assert(KS == 1 || (KS == 2 && TA % 2 == 0), "k-halves: even row tiles");
  // KS = 2: the k-halves' exchange, [4 waves][2 halves][TA/2][TB][64] f32x4
  extern __shared__ __align__(16) float xch_s[];
  int mt0, nt0;
  if ((EPI == EPI_MOD || EPI == EPI_BIAS_SILU) && g.m_dev) {
    // row count known on the device only (usually one panel): panel-major over
    // the XCDs, so that the existing rows' tiles use every CU
    const int tn = g.N / (16 * CT), pm = (int)blockIdx.x / tn;
    mt0 = pm * kBigRowTiles;
    nt0 = ((int)blockIdx.x - pm * tn) * CT;
    g.M = min(g.M, *g.m_dev);
    if (mt0 * 16 >= g.M) return;
  } else if (!big_tile<CT>(g, mt0, nt0)) {
    return;  // whole workgroup: padding of the grid
  }
  // wave index through readfirstlane: scalar per-wave addressing, up to 14 fewer VGPRs
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wq = wave & 3, kh = wave >> 2;  // position in the 2 x 2 wave grid, k-half
  const int wr = wq & 1, wc = wq >> 1;
  const int KB = g.K / kTileK;
  const int nkb = KB / KS;  // this wave's k-blocks kh, kh + KS, ... (the host checks KB % KS == 0)
  const int mt_last = g.m_alloc / 16 - 1;  // allocated row tiles (rows >= M are computed, never stored)
  const op_t *pa[TA], *pb[TB];
#pragma unroll
  for (int i = 0; i < TA; ++i)
    pa[i] = g.A + ((size_t)min(mt0 + wr * TA + i, mt_last) * KB + kh) * kBlockElems + lane * 8;
#pragma unroll
  for (int j = 0; j < TB; ++j) pb[j] = g.W + ((size_t)(nt0 + wc * TB + j) * KB + kh) * kBlockElems + lane * 8;
  constexpr size_t kStep = (size_t)KS * kBlockElems;  // between this wave's consecutive k-blocks
  f16x8 ra[PD][TA], rb[PD][TB];
#pragma unroll
  for (int s = 0; s < PD; ++s) {
    const int kb = min(s, nkb - 1);
#pragma unroll
    for (int i = 0; i < TA; ++i) ra[s][i] = *(const f16x8 *)(pa[i] + kb * kStep);
#pragma unroll
    for (int j = 0; j < TB; ++j) rb[s][j] = *(const f16x8 *)(pb[j] + kb * kStep);
  }
  f32x4 acc[TA][TB];
#pragma unroll
  for (int i = 0; i < TA; ++i)
#pragma unroll
    for (int j = 0; j < TB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < nkb; k0 += PD) {
#pragma unroll
    for (int s = 0; s < PD; ++s) {
      if (k0 + s < nkb) {
#pragma unroll
        for (int i = 0; i < TA; ++i)
#pragma unroll
          for (int j = 0; j < TB; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(rb[s][j], ra[s][i], acc[i][j], 0, 0, 0);
      }
      const int kb = min(k0 + s + PD, nkb - 1);  // past the end: re-load the last block (never used)
#pragma unroll
      for (int i = 0; i < TA; ++i) ra[s][i] = *(const f16x8 *)(pa[i] + kb * kStep);
#pragma unroll
      for (int j = 0; j < TB; ++j) rb[s][j] = *(const f16x8 *)(pb[j] + kb * kStep);
    }
  }

  unsigned bad = 0;  // fp16 range flag of this thread's stores
  if constexpr (KS == 2) {
    // Wave (wq, 0) keeps row tiles [0, H) and hands [H, TA) to wave (wq, 1),
    // which keeps [H, TA); each adds the other's partial of what it keeps.
    constexpr int H = TA / 2;
    f32x4 *xch = (f32x4 *)xch_s;
    f32x4 *mine = xch + (size_t)(wq * 2 + kh) * (H * TB * 64) + lane;
    const f32x4 *other = xch + (size_t)(wq * 2 + (kh ^ 1)) * (H * TB * 64) + lane;
    if (kh == 0) {
#pragma unroll
      for (int i = 0; i < H; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j) mine[(i * TB + j) * 64] = acc[H + i][j];
    } else {
#pragma unroll
      for (int i = 0; i < H; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j) mine[(i * TB + j) * 64] = acc[i][j];
    }
    __syncthreads();
    if (kh == 0) {
#pragma unroll
      for (int i = 0; i < H; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j) acc[i][j] = acc[i][j] + other[(i * TB + j) * 64];
      big_epilogue<EPI, TA, TB, 0, H>(g, acc, mt0 + wr * TA, nt0 + wc * TB, lane, nullptr, bad);
    } else {
#pragma unroll
      for (int i = 0; i < H; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j) acc[H + i][j] = other[(i * TB + j) * 64] + acc[H + i][j];
      big_epilogue<EPI, TA, TB, H, H>(g, acc, mt0 + wr * TA, nt0 + wc * TB, lane, nullptr, bad);
    }
  } else {
    big_epilogue<EPI, TA, TB>(g, acc, mt0 + wr * TA, nt0 + wc * TB, lane, nullptr, bad);
  }
  flush_range(g.status, bad);
}

// LDS-ring kernels of the batched projections: RT x CT 16-row /
// 16-column tiles per workgroup, 8 waves (WR x WC), operands staged through
// an NS-stage LDS ring by LDS-direct loads (RT + CT fragment blocks per
// 32-deep stage).  Each stage's wait is a raw s_barrier after a partial
// vmcnt: __syncthreads' release fence would drain the next stages' loads
// too.  The rows' norm statistics are loaded into registers ahead of the ring
// prologue and folded into rstd after the main loop.  What bounds them (gate/up
// at 3200 rows, 59 us): the LDS-direct fills alone take 34-38 us (16-18 TB/s over
// the chip, 30 bytes per clock and CU, about what L2 hits reach), the products
// alone 41, the waits and barriers of the stages ~10 and the epilogue ~8; 256-row
// tiles and register-pipelined fragments (fewer fills, fewer exposed reads) were
// no faster.  Measured without epilogue (TFLOP/s):
//   gate/up 256 x 128, 4 x 2 waves, 3 stages: 3200 x 8192 x 1024: 800 (vs
//   711 register-streamed), 2048 x 12288 x 1536: 960 (vs 921); with the
//   GeGLU epilogue, 128 x 256 tiles (2 x 4 waves, same LDS per stage) beat
//   256 x 128 in a same-machine A/B: 73.3 -> 66.0 us and 89.3 -> 79.1 us (3200
//   rows are 25 full 128-row panels instead of 12.5 of 256; 800 tiles
//   instead of 832);
//   QKV 128 x 128, 2 x 4 waves, 4 stages: 3200 x 2560 x 1024: 761 (vs 643;
//   at 2048 x 2048 x 1536 the register-streamed kernel stays ahead, 651 vs 621).
// Residual projections on the QKV shape (with epilogue, same-machine A/B against
// the 8-wave k-halves of the register-streamed kernel): 3200 x 1024 x 2048
// 31.1 -> 29.0 us, x 4096 52.6 -> 48.9 us (2 x 4 waves; 4 x 2: 29.9 / 50.7);
// the 1536-wide expert's (2048 rows, 96-column tiles there) lose 5% on
// 128 x 128 ring tiles (192 tiles for 256 CUs) but win on 128 x 96 ones
// (256 tiles, 4 x 2 waves of 32 x 48, 14 fragment blocks per stage): down
// 64.7 -> 62.9 us, O 22.4 -> 21.6 us.
// The wave index goes through readfirstlane so that the compiler keeps the
// per-wave addressing and branches in scalar registers: gate/up on the
// 1536-wide expert 82.1 -> 79.6 us.
constexpr int kRingNW = 8;
template <int EPI>
struct RingShape;
template <>
struct RingShape<EPI_GEGLU> {
  static constexpr int RT = 8, CT = 16, WR = 2, WC = 4, NS = 3;
};
template <>
struct RingShape<EPI_QKV> {
  static constexpr int RT = 8, CT = 8, WR = 2, WC = 4, NS = 4;
};
template <>
struct RingShape<EPI_RESID_F32> {
  static constexpr int RT = 8, CT = 8, WR = 2, WC = 4, NS = 4;
};

// 144 x 256 gate/up tiles, 1 x 8 waves of 144 x 32 (one gate/up pair each):
// fewer tiles where 128-row ones would leave some CUs a fourth tile
struct RingGeGlu144 {
  static constexpr int RT = 9, CT = 16, WR = 1, WC = 8, NS = 3;
};
// 160 x 256 gate/up tiles, 2 x 4 waves of 80 x 64 (two stages at any K: two
// workgroups' three stages and row statistics exceed the 160 KiB of LDS)
struct RingGeGlu160 {
  static constexpr int RT = 10, CT = 16, WR = 2, WC = 4, NS = 2;
};

// Tiles for a few hundred rows, where 128-row tiles leave CUs idle: 64 x 64 (2 x 4
// waves of 32 x 16), 64 x 128 (32 x 32) and, for gate/up, 128 x 128 (64 x 32)
struct Ring64x64 {
  static constexpr int RT = 4, CT = 4, WR = 2, WC = 4, NS = 4;
};
struct Ring64x128 {
  static constexpr int RT = 4, CT = 8, WR = 2, WC = 4, NS = 4;
};
struct Ring128x128 {
  static constexpr int RT = 8, CT = 8, WR = 2, WC = 4, NS = 4;
};

// 128 x 96 tiles: the residual projections where 96-column tiles are preferred
struct RingResid96 {
  static constexpr int RT = 8, CT = 6, WR = 4, WC = 2, NS = 4;
};

// Wait until this wave's loads of all but the newest `later` stages (L
// LDS-direct loads each) have landed, then meet the workgroup.
template <int L>
__device__ __forceinline__ void ring_wait(int later) {
  if (later >= 2)
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * L) : "memory");
  else if (later == 1)
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(L) : "memory");
  else
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <int EPI, int NS = RingShape<EPI>::NS, class S = RingShape<EPI>, bool KSPLIT = false>
__global__ __launch_bounds__(512) void gemm_ring_kernel(GemmArgs g) {
  static_assert(!KSPLIT || EPI == EPI_RESID_F32, "split-K: residual projections");
  constexpr int RT = S::RT, CT = S::CT, WR = S::WR, WC = S::WC;
  // NBLK fragment blocks per stage over the 8 waves: the first NFULL waves
  // issue LPW LDS-direct loads per stage, the others LPW - 1
  constexpr int NBLK = RT + CT, LPW = (NBLK + kRingNW - 1) / kRingNW, NFULL = NBLK - (LPW - 1) * kRingNW;
  constexpr int TA = RT / WR, TB = CT / WC;            // 16 x 16 tiles per wave
  constexpr int ROWS = 16 * RT, TPR = 512 / ROWS;       // rows per workgroup, threads per row's statistics
  static_assert(WR * WC == kRingNW && RT % WR == 0 && CT % WC == 0 && NS >= 2 && NS <= 4, "ring shape");
  typedef __attribute__((address_space(3))) void lds_void;
  extern __shared__ __align__(16) unsigned char ring_smem[];
  op_t *stage = (op_t *)ring_smem;  // [NS][NBLK][512]
  __shared__ float rpart[TPR][ROWS];
  __shared__ float rstd_s[ROWS];
  // split-K: the grid is kx copies of the tile grid, copy `split` taking the
  // split-th of kx equal k-ranges
  const int kx = KSPLIT ? g.kx : 1;
  const int tn = g.N / (16 * CT), per_split = grid_tile_wgs(g.M, ROWS, tn);
  const int split = KSPLIT ? (int)blockIdx.x / per_split : 0;
  int pm, pn;
  if (!grid_tile_at((int)blockIdx.x - split * per_split, g.M, ROWS, tn, pm, pn)) return;  // whole workgroup
  const int mt0 = pm * RT, nt0 = pn * CT;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = wave % WR, wc = wave / WR;
  const int KBt = g.K / kTileK;  // k-blocks of a row
  const int kb0 = split * KBt / kx, KB = (split + 1) * KBt / kx - kb0;  // this workgroup's k-blocks
  const int mt_last = g.m_alloc / 16 - 1;

  auto issue = [&](int kb, int buf) {
    op_t *dst = stage + (size_t)buf * NBLK * kBlockElems;
#pragma unroll
    for (int q = 0; q < LPW; ++q) {
      const int bidx = wave + q * kRingNW;
      if (NFULL < kRingNW && q == LPW - 1 && wave >= NFULL) break;
      const op_t *src = bidx < RT ? g.A + ((size_t)min(mt0 + bidx, mt_last) * KBt + kb0 + kb) * kBlockElems
                                  : g.W + ((size_t)(nt0 + bidx - RT) * KBt + kb0 + kb) * kBlockElems;
      __builtin_amdgcn_global_load_lds((const void *)(src + lane * 8), (lds_void *)(dst + bidx * kBlockElems), 16, 0,
                                       0);
    }
  };
  // per-row sums of squares: TPR threads share row (tid % ROWS), each summing a
  // slice of its partial sums.  The first kPre go out ahead of the ring's loads,
  // so that their use waits for none of those.
  constexpr bool kNorm = EPI != EPI_RESID_F32;
  constexpr int kPre = kNorm ? 16 : 1;  // 64 sums (small-M producer) over 4 threads
  float pre[kPre];
  int t0 = 0, t1 = 0;
  const float *sp = g.ssq;
  const bool norm = kNorm && g.use_rstd && (TPR * ROWS == 512 || (int)threadIdx.x < TPR * ROWS);
  if (norm) {
    const int part = threadIdx.x / ROWS;
    sp += min(mt0 * 16 + (int)(threadIdx.x % ROWS), g.M - 1);
    t0 = part * g.ssq_tiles / TPR;
    t1 = (part + 1) * g.ssq_tiles / TPR;
#pragma unroll
    for (int q = 0; q < kPre; ++q) pre[q] = sp[(size_t)min(t0 + q, g.ssq_tiles - 1) * g.m_alloc];
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (s < KB) issue(s, s);
  __builtin_amdgcn_sched_barrier(0);

  if (norm) {
    float ss = 0.f;
#pragma unroll
    for (int q = 0; q < kPre; ++q) ss += t0 + q < t1 ? pre[q] : 0.f;
    for (int q = t0 + kPre; q < t1; ++q) ss += sp[(size_t)q * g.m_alloc];
    rpart[threadIdx.x / ROWS][threadIdx.x % ROWS] = ss;
  }

  f32x4 acc[TA][TB];
#pragma unroll
  for (int i = 0; i < TA; ++i)
#pragma unroll
    for (int j = 0; j < TB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int kb = 0; kb < KB; ++kb) {
    // stage kb landed for this wave (later stages may stay in flight), then
    // for every wave; the buffer refilled below was last read one step ago
    const int later = min(NS - 2, KB - 1 - kb);  // stages issued after kb
    if (NFULL == kRingNW || wave < NFULL)
      ring_wait<LPW>(later);
    else
      ring_wait<LPW - 1>(later);
    if (kb + NS - 1 < KB) issue(kb + NS - 1, (kb + NS - 1) % NS);
    const op_t *sb = stage + (size_t)(kb % NS) * NBLK * kBlockElems + lane * 8;
    f16x8 af[TA], bf[TB];
#pragma unroll
    for (int i = 0; i < TA; ++i) af[i] = *(const f16x8 *)(sb + (wr * TA + i) * kBlockElems);
#pragma unroll
    for (int j = 0; j < TB; ++j) bf[j] = *(const f16x8 *)(sb + (RT + wc * TB + j) * kBlockElems);
#pragma unroll
    for (int i = 0; i < TA; ++i)
#pragma unroll
      for (int j = 0; j < TB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bf[j], af[i], acc[i][j], 0, 0, 0);
  }

  if constexpr (KSPLIT) {
    // Partial tiles, fp32, [tile][split][wave][i][j][component][lane]: the
    // last workgroup of a tile to arrive adds them in split order, whatever
    // the arrival order, and runs the epilogue; the others are done, and no
    // workgroup waits on another.  The partials are written and read with
    // device-coherent (agent-scope) stores and loads, which bypass the
    // per-XCD L2, so no cache-wide write-back or invalidation is needed: the
    // stores are complete (vmcnt) before the workgroup's arrival is counted.
    __shared__ unsigned kx_last;
    constexpr int PW = TA * TB * 4 * 64;  // floats per wave
    const int tile = pm * tn + pn;
    float *ws = g.kx_ws + (size_t)tile * kx * kRingNW * PW + (size_t)wave * PW + lane;
#pragma unroll
    for (int i = 0; i < TA; ++i)
#pragma unroll
      for (int j = 0; j < TB; ++j)
#pragma unroll
        for (int c = 0; c < 4; ++c)
          __hip_atomic_store(ws + (size_t)split * kRingNW * PW + ((i * TB + j) * 4 + c) * 64, acc[i][j][c],
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0)
      kx_last = __hip_atomic_fetch_add(g.kx_cnt + tile, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                (unsigned)(kx - 1);
    __syncthreads();
    if (!kx_last) return;
    f32x4 own[TA][TB];
#pragma unroll
    for (int i = 0; i < TA; ++i)
#pragma unroll
      for (int j = 0; j < TB; ++j) own[i][j] = acc[i][j];
    for (int sp = 0; sp < kx; ++sp) {
      const float *src = ws + (size_t)sp * kRingNW * PW;
#pragma unroll
      for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j) {
          f32x4 v = own[i][j];
          if (sp != split)
#pragma unroll
            for (int c = 0; c < 4; ++c)
              v[c] = __hip_atomic_load(src + ((i * TB + j) * 4 + c) * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          acc[i][j] = sp == 0 ? v : acc[i][j] + v;
        }
    }
    if (threadIdx.x == 0) __hip_atomic_store(g.kx_cnt + tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }

  if (g.use_rstd) {
    __syncthreads();  // rpart complete (also past every wave's last LDS read of the ring)
    if (threadIdx.x < ROWS) {
      float ss = 0.f;
#pragma unroll
      for (int p = 0; p < TPR; ++p) ss += rpart[p][threadIdx.x];
      rstd_s[threadIdx.x] = 1.0f / sqrtf(ss / (float)g.K + g.eps);
    }
    __syncthreads();
  }
  unsigned bad = 0;  // fp16 range flag of this thread's stores
  if constexpr (EPI == EPI_RESID_F32) {
    // one sum of squares per row of the tile: the wave columns' sums meet in LDS
    static_assert(WC <= TPR, "a row of rpart per wave column");
    big_epilogue<EPI, TA, TB>(g, acc, mt0 + wr * TA, nt0 + wc * TB, lane, nullptr, bad, rpart[wc], mt0 * 16);
    __syncthreads();
    if ((int)threadIdx.x < min(ROWS, g.M - mt0 * 16)) {
      float ss = 0.f;
#pragma unroll
      for (int q = 0; q < WC; ++q) ss += rpart[q][threadIdx.x];
      g.ssq[(size_t)pn * g.m_alloc + mt0 * 16 + threadIdx.x] = ss;
    }
  } else {
    big_epilogue<EPI, TA, TB>(g, acc, mt0 + wr * TA, nt0 + wc * TB, lane,
                              g.use_rstd ? rstd_s + wr * TA * 16 : nullptr, bad);
  }
  flush_range(g.status, bad);
}


template <int EPI, int NS, class S = RingShape<EPI>, bool KSPLIT = false>
static hipError_t launch_ring_ns(const GemmArgs &g, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  const int wgs = grid_tile_wgs(g.M, 16 * S::RT, g.N / (16 * S::CT)) * (KSPLIT ? g.kx : 1);
  const uint32_t lds = (uint32_t)(NS * (S::RT + S::CT) * kBlockElems * sizeof(op_t));
  UAD_LAUNCH((gemm_ring_kernel<EPI, NS, S, KSPLIT>), dim3(wgs), dim3(512), lds, s, ev0, ev1, g);
  return hipGetLastError();
}

// Gate/up on 256-column tiles with K <= 1024: a 2-stage ring (48 KiB of LDS):
// same-machine at 3200 x 8192 x 1024 58.7 us against 61.5 with 3 stages; at
// K = 1536 (2048 x 12288) 2 stages lost 84.2 -> 92.6 us, so 3 there.
static hipError_t launch_ring_geglu(const GemmArgs &g, const ProjRoute &r, hipStream_t s, hipEvent_t ev0,
                                    hipEvent_t ev1) {
  if (r.rows == 64) return launch_ring_ns<EPI_GEGLU, Ring64x128::NS, Ring64x128>(g, s, ev0, ev1);
  if (r.cols == 128) return launch_ring_ns<EPI_GEGLU, Ring128x128::NS, Ring128x128>(g, s, ev0, ev1);
  if (r.rows == 160) return launch_ring_ns<EPI_GEGLU, 2, RingGeGlu160>(g, s, ev0, ev1);
  if (r.rows == 144) {
    if (g.K <= 1024) return launch_ring_ns<EPI_GEGLU, 2, RingGeGlu144>(g, s, ev0, ev1);
    return launch_ring_ns<EPI_GEGLU, RingGeGlu144::NS, RingGeGlu144>(g, s, ev0, ev1);
  }
  if (g.K <= 1024) return launch_ring_ns<EPI_GEGLU, 2>(g, s, ev0, ev1);
  return launch_ring_ns<EPI_GEGLU, RingShape<EPI_GEGLU>::NS>(g, s, ev0, ev1);
}

static hipError_t launch_ring_qkv(const GemmArgs &g, const ProjRoute &r, hipStream_t s, hipEvent_t ev0,
                                  hipEvent_t ev1) {
  if (r.cols == 64) return launch_ring_ns<EPI_QKV, Ring64x64::NS, Ring64x64>(g, s, ev0, ev1);
  if (r.rows == 64) return launch_ring_ns<EPI_QKV, Ring64x128::NS, Ring64x128>(g, s, ev0, ev1);
  return launch_ring_ns<EPI_QKV, RingShape<EPI_QKV>::NS>(g, s, ev0, ev1);
}

template <class S>
static hipError_t launch_ring_resid(const GemmArgs &g, const ProjRoute &r, hipStream_t s, hipEvent_t ev0,
                                    hipEvent_t ev1) {
  if (r.kx == 1) return launch_ring_ns<EPI_RESID_F32, S::NS, S>(g, s, ev0, ev1);
  GemmArgs gk = g;
  gk.kx = r.kx;
  return launch_ring_ns<EPI_RESID_F32, S::NS, S, true>(gk, s, ev0, ev1);
}

template <int EPI, int NS, class S = RingShape<EPI>, bool KSPLIT = false>
static hipError_t ring_attr_ns() {
  return hipFuncSetAttribute((const void *)gemm_ring_kernel<EPI, NS, S, KSPLIT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             NS * (S::RT + S::CT) * kBlockElems * (int)sizeof(op_t));
}

// LDS of the k-halves' exchange (gemm_big_kernel with KS = 2)
template <int CT>
constexpr size_t big_xch_bytes() { return (size_t)4 * 2 * (kBigRowTiles / 4) * (CT / 2) * 64 * sizeof(f32x4); }

template <int EPI, int CT>
static hipError_t launch_big_ct(const GemmArgs &g, const ProjRoute &r, hipStream_t s, hipEvent_t ev0,
                                hipEvent_t ev1) {
  const int wgs = grid_tile_wgs(g.M, 16 * kBigRowTiles, g.N / (16 * CT));
  if constexpr (EPI != EPI_MOD) {
    if (r.halves) {
      UAD_LAUNCH((gemm_big_kernel<EPI, CT, 2>), dim3(wgs), dim3(512), (uint32_t)big_xch_bytes<CT>(), s,
                 ev0, ev1, g);
      return hipGetLastError();
    }
  }
  UAD_LAUNCH((gemm_big_kernel<EPI, CT>), dim3(wgs), dim3(256), 0, s, ev0, ev1, g);
  return hipGetLastError();
}

// What the rules of routes.h see of a launch.
static Proj proj_of(int epi, const GemmArgs &g) {
  Proj p{};
  p.n_cu = g_n_cu; p.epi = epi; p.M = g.M; p.N = g.N; p.K = g.K; p.second = g.A2 != nullptr;
  if (epi == EPI_QKV) p.q_dim = g.q_dim;
  if (epi == EPI_RESID_F32) {
    p.gate = g.mod_gate != nullptr; p.mod_row = g.mod_row != nullptr; p.scale_next = g.mod_scale_next != nullptr;
    if (g.kx_ws && g.kx_cnt) { p.kx_ws_bytes = g.kx_ws_bytes; p.kx_tiles = g.kx_tiles; }
  }
  return p;
}

int resid_ssq_tiles(const GemmArgs &g) { return ssq_tiles_of(proj_of(EPI_RESID_F32, g)); }

template <int EPI, int CT>
static hipError_t big_attr() {
  return hipFuncSetAttribute((const void *)gemm_big_kernel<EPI, CT, 2>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)big_xch_bytes<CT>());
}

hipError_t gemm_init() {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&g_n_cu, hipDeviceAttributeMultiprocessorCount, dev);
  if (e == hipSuccess && g_n_cu < 1) e = hipErrorInvalidDevice;
  if (e == hipSuccess) e = ring_attr_ns<EPI_GEGLU, RingShape<EPI_GEGLU>::NS>();
  if (e == hipSuccess) e = ring_attr_ns<EPI_GEGLU, 2>();
  if (e == hipSuccess) e = ring_attr_ns<EPI_GEGLU, 2, RingGeGlu144>();
  if (e == hipSuccess) e = ring_attr_ns<EPI_GEGLU, RingGeGlu144::NS, RingGeGlu144>();
  if (e == hipSuccess) e = ring_attr_ns<EPI_GEGLU, 2, RingGeGlu160>();
  if (e == hipSuccess) e = ring_attr_ns<EPI_GEGLU, Ring64x128::NS, Ring64x128>();
  if (e == hipSuccess) e = ring_attr_ns<EPI_GEGLU, Ring128x128::NS, Ring128x128>();
  if (e == hipSuccess) e = ring_attr_ns<EPI_QKV, RingShape<EPI_QKV>::NS>();
  if (e == hipSuccess) e = ring_attr_ns<EPI_QKV, Ring64x128::NS, Ring64x128>();
  if (e == hipSuccess) e = ring_attr_ns<EPI_QKV, Ring64x64::NS, Ring64x64>();
  if (e == hipSuccess) e = ring_attr_ns<EPI_RESID_F32, RingShape<EPI_RESID_F32>::NS>();
  if (e == hipSuccess) e = ring_attr_ns<EPI_RESID_F32, Ring64x64::NS, Ring64x64>();
  if (e == hipSuccess) e = ring_attr_ns<EPI_RESID_F32, Ring64x64::NS, Ring64x64, true>();
  if (e == hipSuccess) e = ring_attr_ns<EPI_RESID_F32, RingResid96::NS, RingResid96>();
  if (e == hipSuccess) e = ring_attr_ns<EPI_RESID_F32, RingShape<EPI_RESID_F32>::NS, RingShape<EPI_RESID_F32>, true>();
  if (e == hipSuccess) e = ring_attr_ns<EPI_RESID_F32, RingResid96::NS, RingResid96, true>();
  if (e == hipSuccess) e = big_attr<EPI_BIAS_SILU, 8>();
  if (e == hipSuccess) e = big_attr<EPI_RESID_F32, 6>();
  return e;
}

// Launch shape.  Row groups: up to four 16-row tiles each; when the rows fit
// in four tiles they are spread over more groups (see below).  K: runs of
// KPW = 4 k-blocks per wave, <= 8 waves, as many passes as needed.
GemmPlan plan_gemm(int epi, int M, int N, int K) {
  GemmPlan p{};
  const int KB = K / kTileK;
  p.T = (epi == EPI_GEGLU || epi == EPI_MOD) ? 2 : 1;
  const int ngroups = N / kTileN / p.T;
  const int MT = (M + 15) / 16;
  if (MT > kMaxTilesPerGroup) {
    p.mgroups = (MT + kMaxTilesPerGroup - 1) / kMaxTilesPerGroup;
  } else {
    // small M: spread the row tiles over up to ~1.5 workgroups per CU (each
    // extra group re-reads the weight tile from L2 but halves the activation
    // rows per workgroup; measured best at batch 1: O and down 4 groups,
    // QKV 2-3, gate/up 1)
    const int want = 384 / ngroups;
    p.mgroups = want < MT ? want : MT;
    if (p.mgroups < 1) p.mgroups = 1;
  }
  p.kpw = (KB % 4 == 0) ? 4 : (KB % 2 == 0 ? 2 : 1);
  p.waves = KB / p.kpw < 8 ? KB / p.kpw : 8;
  while (p.waves > 1 && KB % (p.kpw * p.waves) != 0) --p.waves;
  p.passes = KB / (p.kpw * p.waves);
  // every row group must hold 1..4 tiles
  const int max_tiles = (MT + p.mgroups - 1) / p.mgroups;
  p.ok = KB >= 1 && N % (kTileN * p.T) == 0 && p.waves >= 1 && KB == p.passes * p.kpw * p.waves &&
         max_tiles <= kMaxTilesPerGroup && p.mgroups <= MT;
  return p;
}

#define UAD_GEMM_KPW_CASES(EPI, T)                            \
  switch (p.kpw) {                                            \
    case 1: return launch_t<EPI, T, 1>(g, p, s, ev0, ev1);    \
    case 2: return launch_t<EPI, T, 2>(g, p, s, ev0, ev1);    \
    case 4: return launch_t<EPI, T, 4>(g, p, s, ev0, ev1);    \
  }                                                           \
  return hipErrorInvalidValue;

hipError_t launch_gemm(int epi, const GemmArgs &g, const GemmPlan &p, hipStream_t s, hipEvent_t ev0,
                       hipEvent_t ev1) {
  if (g.m_alloc < g.M || g.m_alloc % 16 != 0) return hipErrorInvalidValue;  // operand rows allocated
  const ProjRoute r = route_projection(proj_of(epi, g));
  if (r.kernel == PROJ_RING) {
    switch (epi) {
      case EPI_GEGLU: return launch_ring_geglu(g, r, s, ev0, ev1);
      case EPI_QKV: return launch_ring_qkv(g, r, s, ev0, ev1);
      case EPI_RESID_F32:
        if (r.rows == 64) return launch_ring_resid<Ring64x64>(g, r, s, ev0, ev1);
        if (r.cols == 96) return launch_ring_resid<RingResid96>(g, r, s, ev0, ev1);
        return launch_ring_resid<RingShape<EPI_RESID_F32>>(g, r, s, ev0, ev1);
    }
    return hipErrorInvalidValue;
  }
  if (r.kernel == PROJ_STREAMED) {
    switch (epi) {
      case EPI_BIAS_SILU: return launch_big_ct<EPI_BIAS_SILU, 8>(g, r, s, ev0, ev1);
      case EPI_RESID_F32: return launch_big_ct<EPI_RESID_F32, 6>(g, r, s, ev0, ev1);
      case EPI_MOD: return launch_big_ct<EPI_MOD, 8>(g, r, s, ev0, ev1);
    }
    return hipErrorInvalidValue;
  }
  if (!p.ok) return hipErrorInvalidValue;
  switch (epi) {
    case EPI_BIAS_SILU: UAD_GEMM_KPW_CASES(EPI_BIAS_SILU, 1)
    case EPI_RESID_F32: UAD_GEMM_KPW_CASES(EPI_RESID_F32, 1)
    case EPI_GEGLU: UAD_GEMM_KPW_CASES(EPI_GEGLU, 2)
    case EPI_QKV: UAD_GEMM_KPW_CASES(EPI_QKV, 1)
    case EPI_MOD: UAD_GEMM_KPW_CASES(EPI_MOD, 2)
  }
  return hipErrorInvalidValue;
}

}  // namespace uad
