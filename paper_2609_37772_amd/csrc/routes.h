// Which kernel and tile a projection takes, and how the attention splits its
// keys: the rules alone, on sizes and the CU count.  No HIP in here, so that the
// rules of any CU count can be checked on a machine without a GPU.
#pragma once

#include <stddef.h>

#include <algorithm>

namespace uad {

constexpr int kTileN = 16;
constexpr int kTileK = 32;
// token rows from which the register-streamed 128-row kernels, the split of the
// large residual tiles and (ada_by_class) the adaptive norms by class apply (the
// ring's smaller tiles go by tile count)
constexpr int kBigM = 256;

enum Epilogue : int {
  EPI_BIAS_SILU = 0,   // out = fp16 silu(acc + bias), fragment order
  EPI_RESID_F32 = 1,   // h = (bias | h) + acc; per-tile sum of squares; next operand fp16(h * gain_next)
  EPI_GEGLU = 3,       // out = fp16 gelu_tanh(rstd*acc_gate) * rstd*acc_up (interleaved gate/up)
  EPI_QKV = 4,         // rstd*acc: q -> bf16 q buffer; k, v -> per-layer K / V^T store
  EPI_MOD = 5,         // adaptive-norm modulations of every norm site (see uad_ctx::mod)
};

// What the rules of a projection go by (see GemmArgs).
struct Proj {
  int n_cu;      // compute units of the device
  int epi, M, N, K;
  int q_dim;     // EPI_QKV
  bool second;   // a second operand (A2)
  bool gate, mod_row, scale_next;  // EPI_RESID_F32: which of the modulations are given
  size_t kx_ws_bytes;  // EPI_RESID_F32: split-K workspace and counters (0: none)
  int kx_tiles;
};

enum ProjKernel : int { PROJ_SMALL, PROJ_STREAMED, PROJ_RING };
struct ProjRoute {
  ProjKernel kernel;
  int rows, cols;  // output tile (PROJ_SMALL: unused)
  int kx;          // PROJ_RING: split over K
  bool halves;     // PROJ_STREAMED: k-halves
};

// Output tiles of rows x cols.
inline int tiles_of(const Proj &g, int rows, int cols) { return (g.M + rows - 1) / rows * (g.N / cols); }

// Residual projections: 96-column tiles when they need fewer 16 x 16 output
// tiles per CU than 128-column ones (1536 wide, 2048 rows: 256 tiles of 48
// instead of 192 tiles of 64 with 64 CUs idle).
inline bool resid_prefers_96(const Proj &g) {
  auto per_cu = [&](int ct) {
    return (tiles_of(g, 128, 16 * ct) + g.n_cu - 1) / g.n_cu * ct;
  };
  return g.N % 96 == 0 && per_cu(6) < per_cu(8);
}

// Residual projections on 128 x 128 ring tiles (after the 64 x 64 ones and the
// splits): from 2560 rows, below that once the tiles fill half the CUs.
inline bool ring_resid_fits(const Proj &g) {
  return (g.M >= 2560 || 2 * tiles_of(g, 128, 128) >= g.n_cu) && g.N % 128 == 0 && !g.second &&
         !resid_prefers_96(g);
}

// Tile of the QKV and gate/up projections on the ring, rows * 1000 + columns, or
// 0 for the small-M kernel.  A tile walks all of K in one workgroup, so at a few
// hundred rows 128-row tiles leave most CUs idle and the rest waiting on their
// own load latency; smaller tiles re-read more of the operands for the same
// products.  Same-machine, us per launch by tile (tiles in brackets; "small" is
// the small-M kernel, "before" what the launch took until then):
//   QKV 1024 -> 2560      64 x 64       64 x 128    128 x 128   small / before
//     200 rows             8.5 (160)    11.6 (80)    14.2 (40)    8.8 /  9.9
//     400                  9.9 (280)    12.0 (140)   14.8 (80)   13.0 / 14.9
//     800                 13.0 (520)    14.6 (260)   15.1 (140)       / 18.3
//     1600                19.0 (1000)   17.8 (500)   20.2 (260)       / 20.2
//     2000                24.4 (1280)   23.6 (640)   22.9 (320)       / 22.9
//   QKV 1536 -> 2048: 384 rows 11.0 (192) 15.5 18.8, before 15.6; 1024 rows 15.2
//     (512) 16.7 19.0, before 23.0; 2048 rows 25.8 (1024) 23.0 21.2, before 23.9
//   gate/up 1024 -> 8192  64 x 128      128 x 128   128 x 256   small / before
//     111 rows            10.9 (128)    12.1 (64)    18.7 (32)    9.8 / 11.4
//     200                 11.8 (256)    12.6 (128)   19.1 (64)   16.8 / 19.5
//     400                 13.9 (448)    13.3 (256)   19.4 (128)       / 21.9
//     800                 25.3 (832)    19.0 (448)   20.5 (224)       / 22.8
//     1050                29.2 (1088)   28.8 (576)   27.3 (288)       / 30.0
//   gate/up 1536 -> 12288: 128 rows 15.7 (192) 17.3 26.7, before 26.3; 640 rows
//     36.4 (960) 27.8 (480) 28.9 (240), before 31.4
inline int ring_tile_qkv(const Proj &g) {
  if (g.second || g.M <= 64 || g.N % 64 != 0 || g.q_dim % 16 != 0) return 0;
  const int t64 = tiles_of(g, 64, 64);
  if (16 * t64 < 9 * g.n_cu) return 0;
  if (4 * t64 <= 11 * g.n_cu || g.N % 128 != 0) return 64064;
  // just past one round of 128 x 128 tiles, and smaller ones fit two a CU
  if (tiles_of(g, 128, 128) > g.n_cu && tiles_of(g, 64, 128) <= 2 * g.n_cu) return 64128;
  return 128128;
}

inline int ring_tile_geglu(const Proj &g) {
  if (g.second || g.M <= 64 || g.N % 128 != 0) return 0;
  const int t = tiles_of(g, 64, 128);
  if (16 * t < 9 * g.n_cu) return 0;
  if (t <= g.n_cu) return 64128;
  return tiles_of(g, 128, 128) <= 2 * g.n_cu || g.N % 256 != 0 ? 128128 : 128256;
}

// The residual projections where 96-column tiles are preferred, on the
// 128 x 96 ring from 1024 rows once its tiles fill 3/4 of the CUs, or with
// a long K.  1536-wide expert, same-machine against the register-streamed kernel
// (us): at 2048 and 1536 rows O 22.4 / 21.8 -> 21.8 / 21.1, unsplit down 65.2 /
// 64.8 -> 63.7 / 62.4; at 1024 rows (128 tiles) down (K = 6144) 60.1 -> 58.1 but O
// (K = 1536) 18.0 -> 19.6.  Short K below 3/4 of the CUs: the 64 x 64 tiles up to
// two a CU, then the register-streamed kernel (1345 to 1408 rows at 1536 columns).
inline bool ring96_fits(const Proj &g) {
  return g.M >= 1024 && (4 * tiles_of(g, 128, 96) >= 3 * g.n_cu || g.K >= 4096) && resid_prefers_96(g) &&
         !g.second && g.K / kTileK >= 1;
}

// The residual projections on 64 x 64 ring tiles (kx: split over K), 0 when they
// don't take them.  Short K (O, time MLP): from 9/16 of the CUs in tiles to two
// tiles a CU.  K >= 4096 (down): fewer tiles, split over K four ways up to 2/3 of
// the CUs and two ways up to 27/32.  Same-machine, us per launch (tiles of 64 x 64):
//   O 2048 -> 1024     800 rows (208) 16.0 -> 13.4, 1050 (272) 19.1 -> 15.2, 1600
//     (400) 20.2 -> 16.5, 2000 (512) 21.6 -> 20.4, 2400 (608) 25.5 -> 25.5; 400
//     rows (112) 9.5 -> 12.9, hence the bounds
//   O 1536 -> 1536     384 (144) 13.7 -> 11.1, 640 (240) 18.3 -> 11.4, 1024 (384)
//     17.0 -> 13.7, 2048 (768) 23.0 -> 23.4
//   down 4096 -> 1024  by splits 1 / 2 / 4: 300 rows (80) 14.1 -> 22.0 / 15.7 / 13.1,
//     400 (112) 15.0 -> 22.0 / 15.8 / 13.0, 600 (160) 20.4 -> 22.3 / 18.4 / 17.0, 800
//     (208) 26.0 -> 22.7 / 18.4 / 20.6, 1050 (272) 23.3 -> 28.5; nothing measured between:
//     833 to 896 rows (224) are past the bound and below 64 tiles of 128 x 128, so on the
//     small-M kernel, probably behind the two-way split
//   down 6144 -> 1536  256 (96) 21.3 -> 31.1 / 20.8 / 15.9, 384 (144) 30.4 -> 31.4 /
//     23.4 / 20.7, 640 (240) 27.5 -> 40.6 / 31.5; 128 (48) 14.8 -> - / 23.6 / 15.8
inline int resid_ring64(const Proj &g) {
  if (g.second || g.M <= 64 || g.N % 64 != 0) return 0;
  const int t = tiles_of(g, 64, 64);
  if (g.K < 4096) return 16 * t >= 9 * g.n_cu && t <= 2 * g.n_cu ? 1 : 0;
  if (16 * t < 5 * g.n_cu || 32 * t > 27 * g.n_cu || t > g.kx_tiles) return 0;
  const int kx = 3 * t <= 2 * g.n_cu ? 4 : 2;
  return (size_t)t * kx * 64 * 64 * sizeof(float) <= g.kx_ws_bytes ? kx : 0;
}

// Split-K of the residual projections on 128-row ring tiles: kx = CUs / tiles (at
// most 4) copies of the tile grid, each over an equal k-range of at least 16
// k-blocks, when the tiles fill at most half the CUs and are at least 64 (90 with
// K < 4096); 1 (no split) otherwise, or when the context gave no workspace or it
// is too small.  With K < 4096 the 64 x 64 tiles come first, so that only widths
// without them (288, 480 and the like: a multiple of 96 but not of 64) split
// here.  Same-machine: down (K = 4096) of the 1024-wide expert at 1600 rows (104
// tiles) 49.8 -> 29.1 us, at 1000 rows 28.1 -> 23.4; of the 1536-wide (K = 6144)
// at 1024 rows (128 tiles of 96 columns) 58.0 -> 36.3.  Tiles filling more than
// half the CUs (one workgroup per CU) split two ways when K >= 4096, two
// co-resident workgroups per CU instead of one: down of the 1536-wide expert at
// 16 environments (256 tiles of 128 x 96) 65.5 -> 54.3 us, step 5.595 -> 5.333
// ms; of the 1024-wide at 64 environments (200 tiles) 45.3 -> 43.4 us; with O and
// the time MLP (K = 1536-2048) split as well the step lost (O 22.1 -> 24.3 us,
// 26.9 -> 30.3 us).
inline int resid_ksplit(const Proj &g, int cols) {
  if (g.second || g.M < kBigM || g.N % cols != 0) return 1;
  const int tiles = tiles_of(g, 128, cols);
  if (tiles < 90 && !(g.K >= 4096 && tiles >= 64)) return 1;
  int kx = std::min(4, g.n_cu / std::max(tiles, 1));
  if (kx == 1 && tiles <= g.n_cu && g.K >= 4096) kx = 2;
  while (kx > 1 && (g.K / kTileK) / kx < 16) --kx;
  const size_t part = (size_t)128 * cols * sizeof(float);
  if (kx > 1 && ((size_t)tiles * kx * part > g.kx_ws_bytes || tiles > g.kx_tiles)) return 1;
  return kx;
}

// Gate/up on the shortest of 128-, 144- and 160-row tiles that fits one round
// of co-resident ring workgroups (two per CU), 128 when none does: the tiles
// past the round ran as a second, mostly single-workgroup wave.  Same-machine,
// 144 rows: 2050 rows (544 -> 480 tiles) 57.1 -> 42.5 us, step 3.484 -> 3.210
// ms; 2300 rows 56.5 -> 42.9 us; 1536-wide at 1408 rows (528 -> 480 tiles,
// K = 1536) 75.8 -> 59.7 us, step 5.089 -> 4.666 ms.  160 rows: 2400 rows
// 56.6 -> 44.6 us, step 3.416 -> 3.203 ms; 2500 rows 56.1 -> 45.4 us;
// 1536-wide at 1536 rows 75.4 -> 61.8 us, step 5.017 -> 4.676 ms.  Where
// every shape exceeds the round the taller tiles lost (3200 rows, 800 -> 736
// tiles of 144: 67.0 -> 69.6 us).
inline int geglu_tile_rows(const Proj &g) {
  const int tn = g.N / 256;
  for (int rows : {128, 144, 160})
    if ((g.M + rows - 1) / rows * tn <= 2 * g.n_cu) return rows;
  return 128;
}

// Whether a launch of the register-streamed kernel takes the k-halves (KS = 2):
// its tiles fill at most one round of CUs (one 4-wave workgroup per CU would leave
// every SIMD a single wave), K >= 1536 and the k-blocks split evenly.  Not for the
// modulations.  Measured on launches that are the ring's now: down of the
// 1536-wide expert (2048 rows) 67.7 -> 65.2 us, O and down of the 1024-wide at
// 3200 rows -2%; at K = 1024 (time-MLP out) 18.8 -> 19.6 us, hence the K bound.
inline bool big_khalves(const Proj &g, int cols) {
  return g.epi != EPI_MOD && tiles_of(g, 128, cols) <= g.n_cu && g.K >= 1536 && (g.K / kTileK) % 2 == 0;
}

// The register-streamed kernel: the time MLP in, the modulations, and the
// residual projections on 96-column tiles that the ring leaves, from kBigM rows
// when there are enough output tiles to fill the chip: each tile runs its whole K
// serially in one workgroup, so with few tiles (and long K) the small-M kernel,
// which splits K over waves, is faster.  The threshold is from a sweep over
// 200..3200 rows when every batched projection ran here (the faster kernel in 49
// of 50 cases, the miss by 6%).
inline bool big_ok(const Proj &g) {
  if (g.epi == EPI_QKV || g.epi == EPI_GEGLU || g.M < kBigM || g.N % 128 != 0) return false;
  if (g.epi == EPI_RESID_F32 && !resid_prefers_96(g)) return false;
  const int tiles = tiles_of(g, 128, 128);
  return tiles >= 90 && !(tiles < 128 && g.K > 4096);
}

// The kernel of a projection.
inline ProjRoute route_projection(const Proj &g) {
  const auto tile = [](int t) { return ProjRoute{t ? PROJ_RING : PROJ_SMALL, t / 1000, t % 1000, 1, false}; };
  if (g.epi == EPI_QKV) return tile(ring_tile_qkv(g));
  if (g.epi == EPI_GEGLU) {
    const int t = ring_tile_geglu(g);
    return tile(t == 128256 ? geglu_tile_rows(g) * 1000 + 256 : t);
  }
  // the ring and register-streamed epilogues gate by modulation row and leave an
  // adaptive next norm to a pass of its own
  if (g.epi == EPI_RESID_F32 && (g.scale_next || (g.gate && !g.mod_row))) return tile(0);
  const int cols = g.epi == EPI_RESID_F32 && resid_prefers_96(g) ? 96 : 128;
  if (g.epi == EPI_RESID_F32) {
    if (const int kx = resid_ring64(g)) return ProjRoute{PROJ_RING, 64, 64, kx, false};
    const int kx = resid_ksplit(g, cols);
    if (kx > 1) return ProjRoute{PROJ_RING, 128, cols, kx, false};
    if (ring96_fits(g)) return tile(128096);
    if (ring_resid_fits(g)) return tile(128128);
  }
  if (!big_ok(g)) return tile(0);
  return ProjRoute{PROJ_STREAMED, 128, cols, 1, big_khalves(g, cols)};
}

// Whether gate/up (d_model to F) of M rows runs on the small-M kernel; second: with
// the adaptive norms' second operand.
inline bool gateup_small(int n_cu, int M, int d, int F, bool second) {
  Proj g{};
  g.n_cu = n_cu; g.epi = EPI_GEGLU; g.M = M; g.N = 2 * F; g.K = d; g.second = second;
  return route_projection(g).kernel == PROJ_SMALL;
}

// Adaptive norms by class, past kBigM rows: the modulations of the step's distinct
// flow times only, and the norms as passes of their own, so that QKV and gate/up
// take one operand.  Up to there the passes (~5 us each) cost more than the second
// operand does, and a schedule computes its conditioning once.  Same-machine, 6
// layers of the 1024-wide expert, us per joint step: 64 environments 2680 -> 1346
// (gate/up 160 -> 56, QKV 60 -> 24, modulations 477 -> 33, two norms 13), 32 1779 ->
// 948, 16 1128 -> 804, 8 759 -> 634, 6 696 -> 612.  kBigM rows exactly (4 row groups of
// the small-M kernel) go by class where gate/up then takes the ring: 4 layers, 4 x 64
// + 1024, us per step and per 10-step schedule by token -> by class: 1024-wide 385 ->
// 322, 3813 -> 3022; 768 270 -> 257, 2690 -> 2394; 512 205 -> 224, 1821 -> 2107; 256 209 ->
// 214, 1820 -> 2023.
inline bool ada_by_class(int n_cu, int M, int d, int F) {
  return M > kBigM || (M == kBigM && !gateup_small(n_cu, M, d, F, false));
}

// Sums of squares per row that the projection leaves for the norm: one per
// output tile of the ring kernels, per wave's columns of the register-streamed
// one, per 16 columns of the small-M one.  The consumers re-read all of them for
// every tile.  Same-machine, 64 -> 8 a row: QKV 28.0 -> 25.0 us and gate/up 65.4 ->
// 59.4 at 3200 rows (64 environments 3.845 -> 3.655 ms per joint step), 96 -> 16:
// gate/up 80.9 -> 72.5 us on the 1536-wide expert (1.836 -> 1.748 ms, 8 layers).
inline int ssq_tiles_of(const Proj &g) {
  const ProjRoute r = route_projection(g);
  return g.N / (r.kernel == PROJ_RING ? r.cols : r.kernel == PROJ_STREAMED ? r.cols / 2 : kTileN);
}

// ---------------------------------------------------------------------------
// Prefix repacking
// ---------------------------------------------------------------------------
// Cuts n_env environments x n_kv_heads x n_blk 32-key blocks into launches whose
// 256-thread workgroups fit a grid (its threads stay below 2^32): whole
// environments, or blocks of one.  f(first environment, environments, first
// block, blocks) returns 0 to go on; the result is its last value.
template <class F>
int for_pack_launches(int n_env, int n_kv_heads, int n_blk, F f) {
  constexpr int most = (1 << 24) - 1;
  const int blks = std::min(n_blk, std::max(1, most / n_kv_heads));
  const int envs = blks < n_blk ? 1 : std::max(1, most / (n_kv_heads * blks));
  for (int e = 0; e < n_env; e += envs)
    for (int q = 0; q < n_blk; q += blks)
      if (const int r = f(e, std::min(envs, n_env - e), q, std::min(blks, n_blk - q))) return r;
  return 0;
}

// ---------------------------------------------------------------------------
// Attention
// ---------------------------------------------------------------------------
// Blocks per chunk (one memory round trip); two chunks are resident (double
// buffer), 2 * NB * 32 * HD * 4 bytes of LDS.
constexpr int attn_chunk_blocks(int head_dim) { return head_dim == 256 ? 2 : 4; }
constexpr int kAttnMaxSplits = 32;  // split-KV partials the merge accepts
constexpr int kAttnMerge8 = 8;      // ... up to which it runs one wave a workgroup

// CUs the attention launch has to leave free for the weight read-ahead of its
// extra workgroups (below that the read-ahead is not issued).
constexpr int kReadAheadMinCus = 32;

// What the attention's rules go by: B environments, chunk H, n_blocks 32-key blocks.
struct AttnSizes {
  int n_cu, group, n_kv_heads, head_dim;  // group: query heads per KV head
  int B, H, n_blocks;
  bool small_gateup;  // gate/up runs on the small-M kernel (attn_splits)
  int qblocks() const { return (group * H + 63) / 64; }  // 64-row query blocks of an (environment, KV head)
};

// The most key splits that any call with these sizes takes: the workspace and
// the limit of the no-allocation step are sized by it.  It fills one round of
// workgroups (256) with query blocks x splits, one chunk (one memory round
// trip) per split when that fits.
inline int attn_splits_max(const AttnSizes &a) {
  const int wgs = a.qblocks() * a.B * a.n_kv_heads;
  const int nb = attn_chunk_blocks(a.head_dim);
  int per = nb;
  if ((long)wgs * ((a.n_blocks + nb - 1) / nb) > 256) {
    for (int sp = std::max(1, 256 / wgs);; --sp) {
      per = (a.n_blocks + sp - 1) / sp;
      const int splits = (a.n_blocks + per - 1) / per;
      if (sp == 1 || a.B * a.H < kBigM ||
          8 * ((a.B * a.n_kv_heads * splits + 7) / 8) * a.qblocks() <= a.n_cu - kReadAheadMinCus)
        break;
    }
  }
  if ((a.n_blocks + per - 1) / per > kAttnMaxSplits) per = (a.n_blocks + kAttnMaxSplits - 1) / kAttnMaxSplits;
  if (per > a.n_blocks) per = a.n_blocks;
  return (a.n_blocks + per - 1) / per;
}

// Key splits of a call and the 32-key blocks of each.  One chunk per split
// while the grid (its groups padded to a multiple of the 8 XCDs) fills at most
// half the CUs: the others read weights ahead.  Beyond that two chunks or more
// per split (longer splits run as two key groups inside the workgroup), as many
// splits as leave kReadAheadMinCus CUs to the read-ahead, without which gate/up
// streams its weights from HBM (~27.5 instead of ~22 us at 300-850 rows).
//
// Gate/up on the small-M kernel (up to 128 rows of the 1024-wide expert, every
// adaptive-norm step by token) gains less from that: as many splits as there may be
// where the merge holds them in its 8-split form, whether or not CUs are left, and one
// chunk per split up to 5/8 of the CUs.  Same-machine, us per joint step of 18 layers,
// as in the other steps -> so (few layers stay in the memory-side cache and say little):
//   at most 8, adaptive norms: 4 x 60 + 816 1941 -> 1912 (6 splits -> 7), 5 x 42 + 700 1847 ->
//     1816 (6 -> 8), 9 x 25 + 501 1924 -> 1890 (5 -> 6), 3 x 48 + 300 1414 -> 1392 (3 -> 6); 8 x 25
//     + 501 1774 -> 1785 (5 -> 6), 3 x 50 + 400 1499 -> 1505 (4 -> 8); nine: 3 x 64 + 1000 1697
//     -> 1730 (7 -> 9)
//   one chunk, 144 and 160 workgroups, adaptive norms: 3 x 32 + 640 1230 -> 1217, 3 x 20 + 816
//     961 -> 948; input: 3 x 32 929 -> 915, 8 x 16 + 512 1041 -> 1027; 168 and 192: 4 x 20 +
//     816 1161 -> 1174, 5 x 25 + 501 1411 -> 1449; input: 2 x 56 + 700 977 -> 988, 7 x 18 + 500
//     1037 -> 1077
// Same-machine, 1024-wide expert of 6 layers, us per joint step, 816 + 50 keys
// (28 blocks), by splits:
//   environments   14     10      7      5      4      3      2      1
//        1         241    247    241    250    255    262    278    311
//        2         350    325    325    334    335    341    357    389
//        3         395    394    358    368    368    373    391    420
//        4         442    453    409    417    417    427    442    464
//        6         599    580    553    499    492    506    513    537
//        8         674    665    601    606    544    548    562    573
//       12         834    832    722    719    715    723    660    672
//       20        1082   1065    888    894    872    859    879    783
inline int attn_splits(const AttnSizes &a, int *bps) {
  const int nb = attn_chunk_blocks(a.head_dim);
  auto grid = [&](int sp) { return 8L * (((long)a.B * a.n_kv_heads * sp + 7) / 8) * a.qblocks(); };
  const int most = attn_splits_max(a);
  int sp = std::min(most, (a.n_blocks + nb - 1) / nb);
  if (a.small_gateup && most <= kAttnMerge8 && grid(most) <= a.n_cu) {
    sp = most;
  } else if (16 * grid(sp) > (a.small_gateup ? 10 : 8) * a.n_cu) {
    sp = std::min(most, (a.n_blocks + 2 * nb - 1) / (2 * nb));
    while (sp > 1 && grid(sp) > a.n_cu - kReadAheadMinCus) --sp;
  }
  *bps = (a.n_blocks + sp - 1) / sp;
  return (a.n_blocks + *bps - 1) / *bps;
}

// Bytes that the extra workgroups of the split merge read ahead below kBigM rows: what
// a lane reads while the merge runs, twice that where more than 16 partials take its
// longer form.  Same-machine, us per joint step of 18 layers, input-conditioned, with
// no bound -> with 480 bytes a lane: 16 splits 24 + 1000 716 -> 691, 14 splits 20 + 816
// 712 -> 687, 48 to 50 + 816 no change (11.8 of 13.6 MB at 48, all at 49); past 16
// splits with 480 and 960: 28 + 1000 712 -> 738, 711; 2 x 32 + 1000 765 -> 787, 766; 10 +
// 1020 738 -> 715, 711.
constexpr size_t merge_read_ahead(int rows_pad, int head_dim, int splits) {
  return (size_t)(rows_pad / 16) * (head_dim / 16) * 64 * (splits > 16 ? 960 : 480);
}

// Whether a launch of n_eh x splits groups and qblocks query blocks streams its
// keys a block at a time.
inline bool attn_streamed(int n_cu, int groups, int qblocks, int bps, int nb) {
  return bps > 2 * nb || (bps > nb && 4 * 8 * ((groups + 7) / 8) * qblocks > 3 * n_cu);
}
// Long splits whose 4-wave workgroups would each have a CU to themselves (one
// wave per SIMD walking the split's blocks, ~1.3 us a block at HD = 256, most of
// it the latency of its read -> MFMA -> softmax chain): 8 waves instead, two key
// groups of four.  The two waves of a SIMD hide each other's chains until the
// LDS reads of their fragments bound them.  Same-machine, attention us per
// layer: 1024-wide expert at 32 / 24 environments 36.5 / 36.3 -> 28.0 / 27.0,
// 8 (with its merge) 27.8 -> 24.6; 1536-wide at 8 / 5 28.7 / 28.0 -> 21.4 /
// 20.5.  Beyond one workgroup per CU two 4-wave ones share a CU already.
inline bool attn_two_groups(int n_cu, int groups, int qblocks, int bps, int nb) {
  return attn_streamed(n_cu, groups, qblocks, bps, nb) && groups * qblocks <= n_cu;
}

}  // namespace uad
