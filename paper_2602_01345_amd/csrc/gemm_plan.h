// Which kernel, tile, K slices and rows per launch a projection of the pruned block (or a prediction head) gets: host
// arithmetic on sizes only, without device code.
#pragma once
#include <algorithm>

#include "epilogue.h"
#include "nova_internal.h"

// Tile of the few-rows kernels for `rows` rows, or rg = 0 where the shared-ring kernels are faster.  norm: for a projection
// that normalises its rows itself (gemm_norm_plan).
//  * A tile of rg groups of eight rows and ng groups of eight features loads (rg + ng) groups and computes rg ng, so of
//    the tiles that give every CU one workgroup the one nearest to a square loads least: the rule is the fewest groups
//    on the busiest CU.  Against the narrowest tile over all rows at once (us, weights from HBM): 64 rows, Nout = 1024,
//    K = 1024 / 4096 64 x 8 3.9 / 8.9 (K cut into four slices), 16 x 16 3.0 / 6.7; 128 rows 64 x 8 4.0 / 10.1 (cut),
//    32 x 16 3.3 / 8.3; 64 rows, Nout = 3072 64 x 16 5.4, 32 x 32 4.9.  Cutting K and adding the slices in a second pass
//    is worth it nowhere any more but for 128 rows of K = 8192 (18.1 against 18.6, not counting what its launch costs
//    behind cold caches) and 48 ... 64 rows of K = 12288 (a block of 64 rows of C = 3072 94.1 against 97.8).
//  * Equal counts: the taller tile, which fetches the weights less often, with a long K or many weights (64 x 32 for
//    32 x 64: 64 rows, K = 2304 into 6912 -1.6 us; 200 rows, C = 1920 = K -2.5; 100 rows, K = 4096, Nout = 1024 32 x 16 6.9,
//    16 x 32 7.8), else the wider one, more rows in flight per weight row (a block of 256 rows of C = 512 26.5, 27.3).
//  * Up to eight rows the weights are all there is to load, and the smallest workgroups stream them best where every CU
//    gets as many of them: one (K = 4096, Nout = 1024, one row: 8 x 16 1.0 us more), with K > 1536 two to four (one row,
//    K = 2048, Nout = 8192: 8 x 16 / 8 x 32 0.6 / 0.9 more; K = 1536, Nout = 6144: 0.1 more / 0.1 less; K = 1024, Nout = 4096:
//    0.3 less / the same).  Uneven, the rule above is better (a block of eight rows of C = 2304: 8 x 16 in place of 288
//    workgroups of 8 x 8 out of K = 2304 / 9216 -1.1 / -3.1 us, 8 x 32 in place of 864 -1.5; C = 1920, 8 x 32 in place of 960
//    -0.9).  They have eight waves with K > 2048 (one / eight rows, K = 3072: -0.5 / 0 against four, K = 6144 -1.0 / -0.2, but
//    K = 2048, Nout = 8192 +1.3 / +0.9).
//  * One workgroup per CU beats the 128- and 256-row tiles at any row count (1024 rows, Nout = 1024: K = 1024 8.4
//    against 11.1 us, K = 4096 16.4 against 22.9; 640 rows 7.4 / 14.7 against 11.0 / 17.3).  Two per CU do up to 512 rows
//    (512 rows, K = 1024, Nout = 3072: 10.2 against 10.5; 820 rows, Nout = 1920 = K: 17.8 against 17.2), but not with a
//    long K (400 rows, K = 9216, Nout = 2304: 30 against 27).
//  * A tile's rows of 2 K bytes are addressed with 32-bit offsets: 64 of them up to K = 2^23, 8 up to 2^26 (the down
//    projection of 64 features, K = 2^23 + 2048, 5 / 200 rows: 3.9 / 4.4 ms, 256 x 128 tiles in K slices 20.5 / 25.7).
// The kernels: groups of eight rows, of eight features, waves, units in flight per wave, workgroups that fit a CU.
#define NOVA_ROWS_TILES(T)                                                          \
  T(1, 1, 4, 4, 2) T(1, 1, 8, 4, 2) T(1, 2, 4, 4, 2) T(1, 4, 4, 4, 2) T(2, 1, 4, 4, 2) \
  T(2, 2, 4, 4, 2) T(2, 4, 4, 3, 2) T(4, 2, 4, 3, 2) T(4, 4, 4, 2, 2) T(4, 8, 4, 2, 1) \
  T(8, 4, 4, 2, 1) T(8, 8, 4, 2, 1) T(8, 8, 4, 1, 2)
inline RowsPlan gemm_rows_plan(int num_cus, int mode, int rows, int Nout, int K, bool norm = false) {
  RowsPlan best = {};
  if (mode == EPI_ENTROPY || Nout % 64 != 0) return best;
  const bool weights_only = !norm && rows <= 8 && (Nout <= 8 * num_cus || (K > 1536 && Nout % (8 * num_cus) == 0 && Nout <= 32 * num_cus));
  const bool tall = K >= 4096 || (K >= 1536 && Nout >= 1536);
  const int max_per_cu = mode == EPI_RESIDUAL || rows > 512 ? 1 : 2;
  int64_t least = INT64_MAX;
  auto consider = [&](const RowsPlan& t, int fit) {
    if ((int64_t)std::max(t.rg, t.ng) * 16 * K > 1 << 30) return;                    // see the last rule above
    if (t.rg * t.ng == 1 ? norm || t.kw != (K > 2048 ? 8 : 4) : weights_only) return;       // a long K over twice the waves
    const int64_t wgs = (int64_t)((rows + 8 * t.rg - 1) / (8 * t.rg)) * (Nout / (8 * t.ng));
    const int64_t per_cu = (wgs + num_cus - 1) / num_cus;
    if (rows > 64 && per_cu > std::min(fit, max_per_cu)) return;                     // up to 64 rows: in turns
    const int64_t groups = per_cu * (t.rg + t.ng);
    if (groups < least || (groups == least && (tall ? t.rg > best.rg : t.ng > best.ng))) {
      least = groups;
      best = t;
    }
  };
#define CONSIDER(RG, NG, KW, S, FIT) consider({RG, NG, KW, S}, FIT);
  NOVA_ROWS_TILES(CONSIDER)
#undef CONSIDER
  return best;
}

// Few rows that the projection normalises itself (rg = 0: a launch of its own does it).
//  * Every workgroup normalises its tile's rows again, on one wave per SIMD: some 0.6 us of vector work with 8 rows of 1024, 1.4
//    with 16, against 2.8 us of a launch.  Two norms, us per block in a graph (separate / in the projection): C = 1024 1 row
//    22.4 / 19.6, 8 rows 23.4 / 19.9, 16 rows 26.9 / 26.2, 32 rows 28.0 / 26.6; C = 512 16 rows 22.6 / 19.7, 32 rows 23.2 /
//    21.5; C = 2048 8 rows 39.1 / 35.3, 16 rows 45.7 / 43.4; C = 2560 1 row 47.3 / 45.0, 8 rows 51.9 / 48.2, 16 rows 60.6 / 60.0
//    (QKV alone).  Tiles of 32 rows normalise for 2.5 ... 3.5 us and gain nothing (C = 1024, 36 ... 100 rows: 0 ... +2 us).
//    So tiles of 8 or 16 rows: any projection of up to 8 rows, of up to 16 but for 8192 features and more, which get taller
//    tiles, and of up to 32 of the narrower ones (QKV to C = 1344, up to 1024, cross-attention query to 2048; 256 CUs).
//  * Up to eight rows not the smallest tiles: three or four workgroups per CU would each normalise (C = 2048, 1 / 8 rows
//    37.0 / 39.7 with separate norms, 36.6 / 38.7 with the norm in 768 and 1024 workgroups of 8 x 8, 34.6 / 36.2 in wider tiles).
//    Up projections of more than 8192 features are still 528 ... 640 workgroups of 8 x 16 (C = 2112 ... 2560 above).
//  * A wave holds its rows in registers, 512 elements at a time up to kNormMaxK; a K of 64 per wave at least.
constexpr int kNormMaxGroups = 2, kNormMaxRows = 32, kNormMaxK = 2560;
// Vector of eight elements that a lane reads as its u-th of a row: the row's last one for lanes past its end
constexpr int norm_vector(int u, int lane, int K) { return u * 64 + lane < K / 8 ? u * 64 + lane : K / 8 - 1; }
inline size_t gemm_norm_lds(const RowsPlan& p, int K) { return (size_t)p.rg * 16 * K + (size_t)p.kw * p.s * p.ng * 1024 + 1024; }
inline RowsPlan gemm_norm_plan(int num_cus, int mode, int rows, int Nout, int K) {
  RowsPlan p = {};
  if (rows > kNormMaxRows || K > kNormMaxK) return p;
  if (mode != EPI_QKV && mode != EPI_GELU && mode != EPI_GELU_TANH && mode != EPI_PLAIN) return p;
  p = gemm_rows_plan(num_cus, mode, rows, Nout, K, true);
  if (p.rg > kNormMaxGroups || K < 64 * p.kw) p.rg = 0;
  return p;
}

// Tile configurations (NOVA_GEMM_CFG forces one, for tuning; numbers without a kernel mean 2):
//   1: 256x256x64, 8 waves of 128x64 that alternate between the matrix cores and LDS, or 192x256x64, the same with waves of
//      96x64, where the model prices that lower: more of the CUs busy in a round that 256 x 256 tiles fill by half (us, weights
//      from memory, 256 x 256 or the best plan without it / 192 x 256: 4096 rows, K = 2304, 2304 features 51.2 / 46.0, K = 9216
//      166 / 154; 4915 rows of C = 2048, output 51.1 / 43.8, down 163 / 140; 1229 rows, K = 2304, 9216 features 57.5 / 52.8).
//      Never cut in K: four slices of it lose to slices of the smaller tiles (1046 rows, K = 5632, 1408 features 38.7 / 33.3)
//   2: 256x128x64, 8 waves of 64x64, 3 stages
//   6: 192x128x64, 8 waves of 96x32, 3 stages: one round where 256x128 leaves too many CUs idle and 128x128 needs a
//      second round (1640 rows, K = 1024, 3072 features 17.3 -> 15.7 us; 1100 rows, 4096 features 19.2 -> 16.2)
//   3: 64x32x64, 2 waves of 32x32, 6 stages, staggered K walk          (head entropy only, M <= 64)
//   4: 128x32x64, 4 waves of 32x32, 4 stages, staggered K walk         (head entropy only, M <= 256 or 512)
//   5: 128x128x64, 8 waves of 64x32, 3 stages or, from K = kDeepK on, 4, one workgroup per CU (two waves per SIMD hide the LDS
//      waits that four waves of 64x64 expose: 3-10 % faster at every shape measured).  Three / four stages, us, weights from
//      memory: 900 rows, K = 2304, 2304 features 21.6 / 19.5, 6912 features 44.4 / 42.0; 520 rows, K = 2048, 6144 features
//      20.7 / 19.9; but K = 1536 13.0 / 13.2, K = 1024 10.1 / 10.4 (five: nowhere better than four).  K slices of it have 3
//   7: the few-rows kernels of gemm_rows_bf16.hip (chosen by gemm_rows_plan, not by force)
//   8: 128x64x64, 8 waves of 32x32, 6 stages (with 3: K = 2304 18.6 us in place of 16.3): a narrow output of some 800 ... 2000
//      rows, which 128x128 tiles spread over half of the CUs (us, weights from memory, 128x128 / 128x64: 820 rows, 2304 features
//      out of K = 2304 21.4 / 16.3, 700 rows of 2048 17.9 / 14.5, 1640 rows of 1024 10.4 / 9.4, 2000 rows, K = 2560, 640
//      features 20.4 / 17.2).  A second round of it loses (2458 rows of 1024 10.9 / 17.0)
//   9: 192x256x64 by force (a plan calls it 1; not for a prediction head)
// Without a forced choice the launcher prices 1, 2, 5, 6 and 8 with a model fitted to measurements on MI355X (300 ... 6144
// rows, widths C of 640 ... 2304, outputs of C, 3C and 4C features, K = C and 4C): a launch takes rounds of one tile
// per CU; a round costs a fixed time (first loads, epilogue) and a time per element of K that grows with the share of
// the CUs that are busy (they share L2, memory and power).  The prices of 256x256, 2, 6 and of 5 with three stages at any K are
// fitted for the choice, not for the times, to whole blocks whose weights come from memory as a model's do, with and without
// K slices and in one launch or two: what they chose among themselves was 0.08 % of the block's time from the best on
// average, 4 % at worst (426 sizes; 0.1 % and 7 % on the half of them that a fit leaves out).  192x256 and 8 are priced beside
// them from launches of their own, not in one fit: a block of 160 sizes (513 ... 6000 rows, C = 512 ... 2304) that the two, or
// the fourth stage of 5, change takes 0.972 of its time without on average, 0.89 at best, 1.015 at worst (C = 1600, 4928 rows
// 380 / 386 us; single launches 1.03 at worst: 5984 rows, K = 5376, 1344 features 89.8 / 92.6).  A fit to launches that find
// their weights in L2 makes a single round of 256 x 256 tiles too dear against two of smaller ones, which fetch the weights
// more often: 0.25 %, and blocks up to 7 % slower (1500 rows, C = 1920 / 2048 226 / 237 us, with this one 212 / 228; 1800 rows,
// C = 1024 126 and 120).
constexpr int kNumCfgs = 10;
constexpr int kRowsCfg = 7;
constexpr int kDeepK = 2048;

struct Candidate {
  int cfg, bm, bn;
  double launch, round, gelu;   // us per launch, per round, per round with a GELU
  double k0, k1, k3;            // us per element of K in a round that fills a share f of the CUs: k0 + k1 f + k3 f^3
};

static const Candidate kCands[] = {{1, 256, 256, 3.5, 5.4, 1.8, 0.01806, -0.00115, 0.00630},
                                   {2, 256, 128, 2.4, 3.1, 0.7, 0.00974, -0.00010, 0.00433},
                                   {6, 192, 128, 2.5, 2.7, 0.6, 0.00778, 0.00189, 0.00153},
                                   {5, 128, 128, 2.2, 1.1, 0.1, 0.00649, 0.00120, 0.00165},
                                   {8, 128, 64, 2.2, 2.3, 0.2, 0.00490, 0.00030, 0.00040},
                                   {1, 192, 256, 4.6, 5.3, 1.6, 0.01280, 0.00100, 0.00420}};
inline bool low_tile(const Candidate& c) { return c.cfg == 1 && c.bm == 192; }
// 128 x 64 and the lower height are for projections: a prediction head's rows are many, and full rounds want the 256 x 256
// tile.  A long K leaves 128 x 64 to the tiles that are cut in K: uncut it would gain 2 ... 7 % at 1200 ... 2000 rows of
// K = 4096, 1024 features (2048 rows 30.1 / 28.1 us) and lose elsewhere (820 rows, K = 8192, 2048 features 43.9 / 48.8).
inline bool tile_takes(const Candidate& c, int mode, int K) {
  if (c.cfg == 8) return mode != EPI_ENTROPY && K < 4096;
  return !low_tile(c) || mode != EPI_ENTROPY;
}

// Up to this K the lanes' 32-bit offsets into a tile do: 255 rows of 2 K bytes and the offset along K stay below 2^31.
// Beyond it configuration 2 takes 64-bit addresses, K slices among them, and stands in for 1, 5 and 6; the staggered ones
// (3, 4) of a prediction head always do.  The FFN down projection gets there with few features and a wide FFN.
constexpr int kNearK = 1 << 21;
inline bool tile_fits(int cfg, int K) { return (cfg != 1 && cfg != 5 && cfg != 6 && cfg != 8 && cfg != 9) || K <= kNearK; }
inline bool far_tile(int K) { return K > kNearK; }

// K slices of a launch of `tiles` tiles (the FFN down projection once few tokens are kept: a long K and a narrow
// output fill less than half of the CUs): 2 or 4 workgroups per tile, fp32 partial sums and a second pass.
inline int k_slices(int cus, int mode, int tiles, int64_t rows, int Nout, int K, int64_t part_floats, int forced) {
  if (mode != EPI_RESIDUAL || K < 4096 || forced == 0) return 1;
  int ks = 1;
  if (forced > 0) ks = forced;
  else while (ks < 4 && tiles * ks * 2 <= cus) ks *= 2;
  const bool fits = (ks == 2 || ks == 4) && K % (ks * 64) == 0 && K / (ks * 64) >= 16 && ks * rows * Nout <= part_floats;
  return fits ? ks : 1;
}

// Modelled time (seconds) of one launch over M rows with candidate c.
inline double model_time(const Candidate& c, int slots, int mode, int M, int Nout, int K, int64_t part_floats) {
  const int tiles = ((M + c.bm - 1) / c.bm) * ((Nout + c.bn - 1) / c.bn);
  const int ks = low_tile(c) ? 1 : k_slices(slots, mode, tiles, M, Nout, K, part_floats, -1);
  const int full = tiles * ks / slots, rest = tiles * ks % slots;
  const double f = (double)rest / slots, fixed = c.round + (mode == EPI_GELU || mode == EPI_GELU_TANH ? c.gelu : 0.0);
  double t = c.launch + full * (fixed + K / ks * (c.k0 + c.k1 + c.k3));
  if (rest) t += fixed + K / ks * (c.k0 + c.k1 * f + c.k3 * f * f * f);
  if (ks > 1) t += 2.5 + (ks * 4.0 + 4.0) * M * Nout / 5.9e6;
  // in four slices a launch of 192 x 128 tiles takes either time, at random (60 tiles, K = 6144: 26 or 33 us)
  if (ks == 4 && c.cfg == 6) t += K / ks * 0.0011;
  return t * 1e-6;
}

// Whether M rows of a prediction head go to the narrow-tile kernels (more workgroups for the weight stream).
inline bool narrow_tiles(int M, int Nout, int K) { return M <= 256 || (M <= 512 && Nout < 4096 && K < 4096); }

// Modelled time of the few-rows kernels: what the busiest CU loads at 75 GB/s, half of the weights at the rate of a large
// copy, 2.1 us to start and end (measured 3.0 ... 22 us over 64 ... 1024 rows and 2 ... 38 MB of weights; within 2 us but
// for a long K, where it is up to 8 us too much).
inline double rows_time(const RowsPlan& p, int cus, int rows, int Nout, int K) {
  const int wgs = (rows + 8 * p.rg - 1) / (8 * p.rg) * (Nout / (8 * p.ng));
  const double bytes = (double)((wgs + cus - 1) / cus) * 16.0 * (p.rg + p.ng) * K;
  return 2.1e-6 + bytes / 75e9 + (double)Nout * K / 5e12;
}

inline bool forced_tile(const nova_ctx* ctx) {
  return ctx && ctx->gemm_cfg >= 0 && ctx->gemm_cfg < kNumCfgs && ctx->gemm_cfg != kRowsCfg;
}

// Whether a projection behind a LayerNorm without modulation normalises its rows itself.
inline bool gemm_takes_norm(const nova_ctx* ctx, int mode, int M, int Nout, int K) {
  return !forced_tile(ctx) && gemm_norm_plan(ctx ? ctx->num_cus : 256, mode, M, Nout, K).rg > 0;
}

// Rows of a tile of configuration 1: the height that the model prices lower.
inline int alternating_rows(int slots, int mode, int M, int Nout, int K, int64_t part_floats) {
  int bm = 256;
  double best = 1e30;
  for (const Candidate& c : kCands) {
    if (c.cfg != 1 || !tile_takes(c, mode, K)) continue;
    const double t = model_time(c, slots, mode, M, Nout, K, part_floats);
    if (t < best) { best = t; bm = c.bm; }
  }
  return bm;
}

// Whether a launch of configuration cfg is of 192 x 256 tiles, and whether it can be cut in K.
inline bool low_launch(const nova_ctx* ctx, int cfg, int mode, int rows, int Nout, int K, int64_t part_floats) {
  if (cfg == 9) return true;
  return cfg == 1 && !forced_tile(ctx) && alternating_rows(ctx ? ctx->num_cus : 256, mode, rows, Nout, K, part_floats) == 192;
}
inline bool cut_in_k(int cfg, bool low) { return (cfg == 1 && !low) || cfg == 2 || cfg == 5 || cfg == 6; }

inline int pick_cfg(const nova_ctx* ctx, int mode, int M, int Nout, int K, int64_t part_floats, double* t_out = nullptr) {
  if (forced_tile(ctx)) {
    const bool has = tile_fits(ctx->gemm_cfg, K) && (mode != EPI_ENTROPY || ctx->gemm_cfg < kRowsCfg);
    return has ? ctx->gemm_cfg : 2;
  }
  if (mode == EPI_ENTROPY) {
    if (M <= 64) return 3;
    if (narrow_tiles(M, Nout, K)) return 4;
  }
  const int slots = ctx ? ctx->num_cus : 256;
  const RowsPlan rows = gemm_rows_plan(slots, mode, M, Nout, K);      // rg = 0 for a prediction head
  if (rows.rg) {
    if (t_out) *t_out = rows_time(rows, slots, M, Nout, K);
    return kRowsCfg;
  }
  int best = 2;
  double best_t = 1e30;
  // a prediction head's partials (16 bytes per row and column tile) that fit the static scratch with 256-column tiles
  // only: those, in every entry point, so that the allocation-free one gives the same bits
  const int64_t room = (int64_t)head_entropy_static_capacity() / 16;
  const bool wide = mode == EPI_ENTROPY && (int64_t)M * ((Nout + 127) / 128) > room && (int64_t)M * ((Nout + 255) / 256) <= room;
  for (const Candidate& c : kCands) {
    if (wide && c.bn < 256) continue;
    if (!tile_fits(c.cfg, K) || !tile_takes(c, mode, K)) continue;
    const double t = model_time(c, slots, mode, M, Nout, K, part_floats);
    if (t < best_t) { best_t = t; best = c.cfg; }
  }
  if (t_out) *t_out = best_t;
  return best;
}

// A launch plan: one configuration for all rows, or two launches -- typically (nearly) whole rounds of large
// tiles over the first rows and the best single configuration for the rows left over, so that only a small
// remainder pays for a ragged last round.  Returns the number of parts; part i covers rows [m_base[i], m_end[i]) with cfg[i].
struct Plan {
  int n;
  int m_base[2], m_end[2], cfg[2];
};
inline Plan plan_rows(const nova_ctx* ctx, int mode, int M, int Nout, int K, int64_t part_floats) {
  Plan p;
  double t_single = 1e30;
  p.n = 1; p.m_base[0] = 0; p.m_end[0] = M; p.cfg[0] = pick_cfg(ctx, mode, M, Nout, K, part_floats, &t_single);
  if (forced_tile(ctx) || mode == EPI_ENTROPY || M <= 512 || (ctx && ctx->gemm_parts == 0)) return p;   // one launch
  const int slots = ctx ? ctx->num_cus : 256;
  double best = t_single * 0.97;                          // a second launch has to pay for itself
  for (const Candidate& c : kCands) {
    if (!tile_fits(c.cfg, K) || !tile_takes(c, mode, K)) continue;
    const int tiles_n = (Nout + c.bn - 1) / c.bn;
    for (int rounds = 1;; ++rounds) {                     // rounds of the first part
      const int64_t m1_all = (int64_t)rounds * slots / tiles_n * c.bm;
      if (m1_all >= M) break;
      const int m1 = (int)m1_all;
      if (m1 == 0) continue;
      double t_rest = 0.0;
      const int cfg_rest = pick_cfg(ctx, mode, M - m1, Nout, K, part_floats, &t_rest);
      const double t = model_time(c, slots, mode, m1, Nout, K, part_floats) + t_rest;
      if (t < best) {
        best = t;
        p.n = 2;
        p.m_base[0] = 0; p.m_end[0] = m1; p.cfg[0] = c.cfg;
        p.m_base[1] = m1; p.m_end[1] = M; p.cfg[1] = cfg_rest;
      }
    }
  }
  return p;
}
