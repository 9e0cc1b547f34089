// bf16 GEMM on the CDNA4 matrix cores for the prefill phase (and for decoding batches too wide for
// the streaming kernels):
//   Y[M,N] = act(X[M,K] W[N,K]^T + bias) + residual,  fp32 accumulate.
// Both operands are K-contiguous, so a lane's 8-element MFMA fragment is one
// 16-byte LDS read.  The tile is computed transposed (weight rows as the MFMA
// row operand, activation rows as the column operand).
//
// What bounds the large tiles: power (with N(0,1)-like operands the clock settles at 1.7-1.9 GHz) and, beside it, the
// loads of operand tiles through a compute unit's load path - a 256x256 k-tile of 16384 x 36864 x 12288 takes 1.42 us
// (1.53 with the loop before this one), 1.19 without its 64 KB of loads and 1.30 without its matrix instructions; in a
// launch of one round (4096 x 4096) the loads alone took all of its 1.55 us (these with two stages of weights, not three).
// 32x32x16 instructions, loads and fragment reads in clumps -> 16x16x32, dealt out one by one, 8 x 4 tiles per XCD:
// 16384 x 36864 x 12288 10.85 -> 10.18 ms, 2048 x 15360 x 5120 258 -> 250 us.
// The third stage of weights, two against three in turn: K = 5120: 4096 x 15360 502 -> 482 us, 16384 x 20480 2583 -> 2477
// (3-4 %); K = 9216: 0-1.5 %; K = 12288: none at 4096 rows (x 36864, x 49152), and from 8192 rows on, where power bounds
// the loop, between 0.6 % faster and 1.1 % slower (16384 x 36864 10.15 -> 10.20 ms, x 49152 13.51 -> 13.63; another time
// x 36864 10.04 -> 10.15).  A ring with two stages only for those would be a kernel more for that 1 %.
// What bounds the others: see layer_plan.
//
// Tile BM x BN (activation rows x weight rows, kTiles), BK = 64,
// 256 threads = 4 waves (one per SIMD).  Operands go global -> LDS directly (no register
// staging) into two LDS rings, one per operand (two to four stages), one barrier per k-tile; fragment reads and load issue are
// interleaved with the MFMAs by hand (scheduling fences); the epilogue is
// staged through LDS so bias / residual / output move as 16-byte row pieces.
#include <cmath>

#include "gemm_kernel.h"

namespace ds {

DS_SWITCH(g_gemm_nt, -1);      // 0, 1: never, always
DS_SWITCH(g_gemm_spread, -1);  // 0, 1: never, always

// Weights carry the non-temporal hint where they come from memory once: up to eight row tiles, which an XCD's 32
// workgroups take together (patch_tile).  They leave the activations, which every workgroup reads, in L2: 256 x 49152 x
// 12288 303 -> 241 us, 256 x 12288 x 12288 98 -> 85, 512 x 36864 x 12288 431 -> 377, 256 x 32768 x 8192 171 -> 121.  At
// 12 row tiles it is a draw (2985 x 15360 x 5120 362 and 374 us, x 20480 499 and 479), at 32 the weights are read again
// from further away (8192 x 12288 x 49152 6.98 and 7.79 ms).
//   Small ones are better without it, also where 2.2 GB of other weights come between two uses of theirs.  Each product on
// its plan, without and with the hint: 4096 x 4096 (34 MB) at 128 rows 17.2 and 19.0 us, at 256 22.7 and 24.8, from 275 on
// the same; 5120 x 5120 (52 MB) at 128 rows 23.1 and 24.4, at 160 26.0 and 28.2, from 224 on the same; 12288 x 4096 (101
// MB) at 160 and 256 rows 36.3 and 35.0, 44.1 and 42.1; 8192 x 8192 (134 MB) 43.3 and 38.8, 50.5 and 46.6; 15360 x 5120
// (157 MB) 45.0 and 43.8, 58.9 and 57.9.  (Slower with it above the line: 4096 x 16384 on 11 splits, 224 rows 48 and 55.)
constexpr int kFewRowTiles = 8;
//   That is for the products of a layer, whose other weights come between two uses of these.  ds_linear may be called with
// the same weights again, and the last-level cache holds 256 MB, out of which the hint would keep them: 15360 x 5120 (157
// MB) again and again at 256 / 512 / 1024 / 2048 rows 62 / 86 / 126 / 245 us with the hint, 50 / 73 / 120 / 235 without.
constexpr double kStreamedBytes = 96e6, kCachedBytes = 256e6;

// Workgroups of such launches start at different places of K where the row stride is a multiple of 4 KB (256 x 36864 x
// 12288 215 -> 197 us, 256 x 32768 x 8192 128 -> 112, K of 20480 and 49152: no difference).
static hipError_t launch_tile(int tile, GemmParams p, int splits, bool in_layer, hipStream_t stream) {
  const Tile& t = kTiles[tile];
  p.tiles_m = (p.M + t.bm - 1) / t.bm;
  p.tiles_n = (p.N - p.n_base + t.bn - 1) / t.bn;
  p.splits = splits;
  p.spread = p.K % 2048 == 0;
  if (g_gemm_spread >= 0) p.spread = g_gemm_spread;
  bool nt = p.tiles_m <= kFewRowTiles && 2.0 * p.N * p.K >= (in_layer ? kStreamedBytes : kCachedBytes);
  if (g_gemm_nt >= 0) nt = g_gemm_nt;
  return tile < kFirstLayerTile
             ? launch_any<1>(tile, p, nt, splits, stream, std::make_integer_sequence<int, kFirstLayerTile - 1>())
             : launch_layer_tile(tile, p, nt, splits, stream);
}

// Cost model used to pick a tile shape: (rounds of workgroups on 256 CUs, one workgroup per CU) x
// tile area x a per-area factor of the tile shape.  Under sustained matrix load the chip runs at its
// power limit, so a partly filled last round costs less than a full one (the busy CUs clock higher):
// only 30 % of the idle part of the last round is charged.  Factors are measured ratios of time per
// flop: the 256x256 tile moves 23 % fewer operand bytes per flop than 256x160, the 128x128 tile 50 % more.
static double tile_cost(int M, int N, int BM, int BN, double factor) {
  const long tiles = (long)((M + BM - 1) / BM) * ((N + BN - 1) / BN);
  const double exact = tiles / 256.0;
  const double full = (double)((tiles + 255) / 256);
  const double rounds = tiles <= 256 ? 1.0 : exact + 0.3 * (full - exact);
  return rounds * BM * BN * factor;
}

DS_SWITCH(g_gemm_variant, 0);     // 0 = plan, > 0: force this tile (kTiles)
DS_SWITCH(g_gemm_splits, 0);      // 0 = plan, > 0 force the split count
DS_SWITCH(g_gemm_tail_split, 1);  // 0 = never cut a product at a column
DS_SWITCH(g_gemm_cut_cols, 0);    // > 0: cut at this column ...
DS_SWITCH(g_gemm_tail_kind, 0);   // ... with this tile for the rest

// Tile shape by the cost model above; split count so that a launch with few tiles still occupies the
// chip.  Measured on the decode shapes (M <= 256): >= ~100 workgroups of 128 weight rows stream at
// 5-6 TB/s unsplit; 40 tiles need 4-6 splits; more than ~250 workgroups gain nothing.
// Up to 256 rows the product is bound by streaming the weights, not by the matrix cores, and what a launch
// costs is the bytes its busiest compute unit has to pull through its load path (about 35 GB/s per unit,
// activation re-reads out of L2 included): rounds x (weight + activation bytes of a workgroup's K share
// + its partial tile), plus the reduce pass when K is split.  Used where the rule below would start a second,
// mostly empty round (FFN-in of OPT-13B at 256 rows: 320 tiles of 128x128, 111 us; re-planned 77 us).  For
// single-round launches the measured split counts of the rule below beat this model by 5-25 %, so it is
// not applied to them.
static GemmPlan decode_plan(int M, int N, int K) {
  static const int kBm[5] = {0, 256, 128, 256, 64}, kBn[5] = {0, 160, 128, 256, 128};
  const int kt = K / kBK;
  const int max_s = kt / 8 > 0 ? (kt / 8 < 32 ? kt / 8 : 32) : 1;  // at least 8 k-tiles per split
  GemmPlan best{2, 1};
  double best_cost = 1e30;
  for (int v = 1; v <= 4; ++v) {
    const long tm = (M + kBm[v] - 1) / kBm[v], tn = (N + kBn[v] - 1) / kBn[v];
    const double rows = (double)M / tm;  // activation rows a tile really has
    for (int sp = 1; sp <= max_s; ++sp) {
      const long wgs = tm * tn * sp;
      const double rounds = (double)((wgs + 255) / 256);
      double cost = rounds * ((kBn[v] + rows) * ((double)K / sp) * 2.0 + (sp > 1 ? kBm[v] * kBn[v] * 4.0 : 0.0));
      if (sp > 1) cost += (double)sp * M * N * 4.0 / 256.0 + 175e3;  // reduce pass: its reads, and about 5 us
      if (cost < best_cost) {
        best_cost = cost;
        best = GemmPlan{v, sp};
      }
    }
  }
  return best;
}

// Prefill-sized products (more than 256 rows) of ds_linear, and of a layer from 4097 on: tile shape, split count and
// column cut together, by a time model fitted to this chip (OPT-13B shapes, 512-2048 rows, weights not resident in any cache).
//  * A workgroup's k-loop costs us_per_kk microseconds per 1000 elements of K when all 256 compute units are
//    busy, plus t0 for its prologue and epilogue (the output burst of a whole round of tiles is bound by write
//    bandwidth: 9 us for 256x256 tiles, 5 us for 256x160).
//  * Fewer workgroups than compute units: the busy ones clock higher (the chip is power-limited under matrix
//    load), so only 30 % of the idle share is charged.  A partly filled round after full ones is charged
//    80 % of its idle share: its tiles cost what the full rounds' tiles cost.
//  * Splitting K pays where the tiles alone leave most of the chip idle - 512 to 1024 rows against 5120
//    output columns: FFN-out of OPT-13B at 512 rows 186 -> 118 us on four splits of 256x160 tiles, at 1024
//    rows 357 -> 202 us on two.  It costs the fp32 partials' round trip (cheap while they fit the caches) and
//    a reduce launch, and is only considered for launches that stay within one round.
//  * Tile quantisation: 2.5 rounds cost nearly 3.  A product may be cut at a column: the leading columns keep
//    the large tile in whole rounds, the rest runs as a second launch on 256x160 or 128x128 tiles (bias,
//    residual and output pointers follow the cut).  FFN-in of OPT-13B at 2048 rows: 383 us whole, 348 us as
//    two rounds of 256x256 tiles plus one of 256x160.
// The constants were fitted to the loop with 32x32x16 instructions; from 512 rows up the present one takes 5 % less on
// 256x160 tiles, 4 % on 256x256 and 128x256 (nothing where 256x256 tiles are split), 2 % on 128x128.
// Against every forced tile and split count (512, 1024 and 2048 rows of the OPT-13B, 66B and 175B products) the plans
// are still within 3 % of the fastest, but for one: 512 x 12288 x 12288, 181 us planned, 167 on 128x256 tiles.
struct TileModel {
  int variant, bm, bn;
  double us_per_kk, t0;
};
static const TileModel kTileModels[] = {{3, 256, 256, 24.2, 11.6}, {1, 256, 160, 16.5, 7.9},
                                        {5, 128, 256, 15.0, 8.0}, {2, 128, 128, 11.5, 6.0},
                                        // for the columns behind a cut only: FFN-in of OPT-13B at 2048 rows ends
                                        // on 4096 columns = one exact round of 256x128 tiles (355 us for the
                                        // product against 362 us with 208 tiles of 256x160).  (A 256x224 tile,
                                        // which makes QKV two exact rounds of 8192 + 7168 columns, measured 2 %
                                        // slower than 1.875 rounds of 256x256 tiles: not kept.)
                                        {6, 256, 128, 14.5, 7.0}};
// time of `tiles` workgroups of tile t over K (one launch, no split)
static double tiles_us(const TileModel& t, long tiles, double K) {
  const double exact = tiles / 256.0, full = (double)((tiles + 255) / 256);
  if (tiles <= 256) return (0.7 + 0.3 * exact) * t.us_per_kk * K * 1e-3 + t.t0;
  return (exact + 0.8 * (full - exact)) * (t.us_per_kk * K * 1e-3 + t.t0);
}
static GemmPlan prefill_plan(int M, int N, int K) {
  const int kt = K / kBK;
  GemmPlan best{1, 1};
  double best_us = 1e30;
  for (const TileModel& t : kTileModels) {
    if (t.variant > 5) continue;
    const long tm = (M + t.bm - 1) / t.bm, tn = (N + t.bn - 1) / t.bn;
    const long tiles = tm * tn;
    for (int sp = 1; sp <= 8; ++sp) {
      if (sp > 1 && (kt / sp < 8 || tiles * sp > 256)) break;
      double us = tiles_us(t, tiles * sp, (double)K / sp);
      if (sp > 1) {  // larger fp32 epilogue, a reduce launch, partials out and back
        const double mn = (double)M * N;
        us += 4.0 + 2.0 + (8.0 * sp + 2.0) * mn / (sp * mn * 4.0 <= 32e6 ? 12e6 : 5e6);
      }
      if (us < best_us) {
        best_us = us;
        best = GemmPlan{t.variant, sp};
      }
    }
    if (!g_gemm_tail_split || (t.variant != 1 && t.variant != 3) || tiles <= 256) continue;
    // cut after c column tiles (whole rounds of the large tile only), the rest on a smaller tile
    for (long c = tn - 1; c >= 1; --c) {
      if ((tm * c) % 256 != 0 && tm * c > 256) continue;
      const long rest = N - c * t.bn;
      if (rest <= 0) continue;
      for (const TileModel& u : kTileModels) {
        if (u.variant != 1 && u.variant != 2 && u.variant != 6) continue;
        if (u.variant == 1 && t.variant == 1) continue;
        if (u.bn > t.bn) continue;
        const long tiles_u = (long)((M + u.bm - 1) / u.bm) * ((rest + u.bn - 1) / u.bn);
        const double us = tiles_us(t, tm * c, K) + tiles_us(u, tiles_u, K) + 3.0;  // a second launch
        if (us < best_us) {
          best_us = us;
          best = GemmPlan{t.variant, 1, (int)(c * t.bn), u.variant};
        }
      }
    }
  }
  if (g_gemm_cut_cols > 0 && g_gemm_cut_cols < N) best = GemmPlan{3, 1, g_gemm_cut_cols, g_gemm_tail_kind};
  return best;
}

// The products of a whole layer (layer_plan): every tile, split count and column cut, by a time model.  ds_linear keeps
// the plans above, which are part of what it tells its callers (ds_linear_plan, ds_linear_workspace_bytes).
//
// What bounds a product of some hundred rows is neither the matrix cores nor HBM by itself but what a compute unit gets
// through its load path: its vector memory returns in order, about 106 GB/s out of L2, 51 GB/s (one unit alone) or 26
// (all of them) out of HBM, and 40 to 55 of any mix of the two, whatever is in flight, so a product costs the bytes its
// tiles load.  Those are fewest for one tile over all rows, as wide as registers allow, with K split until the chip is
// full; hence tiles of many heights, and splits that pay for themselves long before the tiles alone fill the chip.  The
// model: a launch of n workgroups takes pl + sqrt(loop^2 + hbm^2) + r (t0) [+ reduce], loop = r (k-tiles of a split)
// k_us, hbm = the weights at 10.7 TB/s (with the square root: what the weights' own stream adds, most where few rows
// leave little else), r = the rounds of 256 workgroups, of which idle units are charged less than busy ones (they leave
// the others power), and 6 % more per k-tile when there are many rounds.  Fitted to 16 products (the four of OPT-13B,
// 66B, 175B and of 8192 x 32768 with 8 of 64 key/value heads), 30 row counts from 65 to 4096 and every tile and split
// that fills more than half the chip, weights not in any cache: its choice is within 1.5 % of the fastest (geometric
// mean; 0.3 % from 1025 rows on).  Against the plans above it saves 27 % of a product's time at 129 to 256 rows (12288 x
// 49152: 461 -> 273 us at 256), 20 % at 257 to 512 (the four of OPT-13B at 275 rows: 283 -> 232 us), 10 % to 1024, 3 %
// to 4096.  More rows are left to the plans above (within 1 % of each other).
//   Four things a second sweep showed (32 products: those and the ones of layers of 1024, 2048 and 4096 features, 38 row
// counts, 2.2 GB of weights in rotation, against the plans above and the ones without these terms):
// kAlone: one row tile over weights without the hint (launch_tile), where its k_us, fitted with it, are short: 5120 x 5120 at
//   208 and 256 rows 29.7 and 31.7 us on 256x128 tiles, 27.4 and 29.7 on 128x128.
// kFewChannels: rows a multiple of 64 KB apart; a multiple of four splits meets fewer memory channels there, turns or not:
//   8192 x 32768 on 128x256 tiles at 96 and 128 rows 104.8 and 111.7 us with 8 splits, 97.7 and 105.7 with 7.  Not with 256x256
//   tiles, whose loads do not bound them (240 rows: 139 us on 8 splits, 145 on 256x192), nor with more row tiles (512 rows: 228
//   on 4 splits, 250 on 2).
// kCut: 57 cuts within 3 % of the best plan without one took 2 % more beside it than the sum of their launches says (median).
//   9216 x 9216 at 2048 rows 279 us cut, 269 not, 12288 x 49152 1897 and 1808; those that pay stay (27648 x 9216 at 2048 rows
//   746 us cut, 797 not).
// kKeep: up to 256 rows of weights without the hint the plan above (most often 128x128 tiles, of which the model has two row
//   tiles 10 to 15 % too long) stays unless another tile promises 10 %: 5120 x 5120 at 160 rows 26.0 -> 25.2 us, 4096 x 4096
//   22.1 -> 20.3.
// What stays slower than without plans of a layer: 65 to 112 rows of 4096 and 2048 features to three times as many (26.7 us
// before, 29.1; 14.3 before, 17.3), where skinny_us is too long for launches that leave units idle.
struct LayerModel {
  static constexpr double kLaunch = 4.8, kIdle = 0.33, kLate = 0.71, kHeat = 0.06;  // us, shares
  static constexpr double kHbm = 10.7e6, kReduce = 4.0, kPartials = 8.7e6;          // bytes a us, us, bytes a us
  static constexpr double kCut = 1.015, kKeep = 0.90;
  static constexpr double kAlone = 0.15, kFewChannels = 0.10;                       // shares
};
static double layer_us(const Tile& t, int rows, int N, int K, int splits) {
  const long tiles_m = (rows + t.bm - 1) / t.bm, tiles = tiles_m * ((N + t.bn - 1) / t.bn) * splits;
  const double exact = tiles / 256.0, full = (double)((tiles + 255) / 256);
  const double rounds = tiles <= 256 ? 1.0 - LayerModel::kIdle * (1.0 - exact) : exact + LayerModel::kLate * (full - exact);
  const double heat = tiles <= 256 ? 1.0 : 1.0 + LayerModel::kHeat * (1.0 - 1.0 / exact);
  double loop = rounds * ((K / kBK + splits - 1) / splits) * t.k_us * heat;
  if (tiles_m == 1 && 2.0 * N * K < kStreamedBytes) loop *= 1.0 + LayerModel::kAlone;
  if (splits % 4 == 0 && K % 32768 == 0 && tiles_m == 1 && t.bm * t.bn < 256 * 256) loop *= 1.0 + LayerModel::kFewChannels;
  const double hbm = 2.0 * N * K / LayerModel::kHbm;
  double us = LayerModel::kLaunch + sqrt(loop * loop + hbm * hbm) + (rounds > 1.0 ? rounds : 1.0) * t.t0_us;
  if (splits > 1) us += LayerModel::kReduce + (8.0 * splits + 2.0) * rows * N / LayerModel::kPartials;
  return us;
}

static GemmPlan gemm_plan(int M, int N, int K);

GemmPlan layer_plan(int M, int N, int K, size_t partial_bytes, double* us_out) {
  const int rows = (M + 31) / 32 * 32, kt = K / kBK;  // by rows in 32s: sizing a workspace asks for every plan up to M
  GemmPlan best{2, 1};
  double best_us = 1e30;
  for (int i = 1; i < kNumTiles; ++i) {
    const Tile& t = kTiles[i];
    const long tm = (rows + t.bm - 1) / t.bm, tn = (N + t.bn - 1) / t.bn;
    for (int sp = 1; sp <= 32; ++sp) {
      if (sp > 1 && (kt / sp < 6 || tm * tn * sp > 256 || sizeof(float) * sp * rows * (size_t)N > partial_bytes)) break;
      const double us = layer_us(t, rows, N, K, sp);
      if (us < best_us) {
        best_us = us;
        best = GemmPlan{i, sp};
      }
    }
    // The last whole rounds of a large tile before a cut; the remaining columns on another tile.
    if (tm * tn <= 256 || t.bm * t.bn < 256 * 192) continue;
    long step = 256;
    while (step > 1 && tm * (step / 2) % 256 == 0) step /= 2;  // columns of tiles that make whole rounds
    const long c = (tn - 1) / step * step;
    if (c == 0) continue;
    const int rest = N - (int)(c * t.bn);
    const double head_us = layer_us(t, rows, (int)(c * t.bn), K, 1);
    for (int j = 1; j < kNumTiles; ++j) {
      if (!kTiles[j].tail || kTiles[j].bn >= t.bn) continue;
      const double us = (head_us + layer_us(kTiles[j], rows, rest, K, 1)) * LayerModel::kCut;
      if (us < best_us) {
        best_us = us;
        best = GemmPlan{i, 1, (int)(c * t.bn), j};
      }
    }
  }
  if (rows > 128 && rows <= 256 && 2.0 * N * K < kStreamedBytes) {
    const GemmPlan own = gemm_plan(rows, N, K);
    const double us = layer_us(kTiles[own.tile], rows, N, K, own.splits);
    if (own.tile != best.tile && best_us > LayerModel::kKeep * us && (own.splits == 1 || sizeof(float) * own.splits * rows * (size_t)N <= partial_bytes)) {
      best_us = us;
      best = own;
    }
  }
  if (us_out) *us_out = best_us;
  best.in_layer = true;
  return best;
}

static GemmPlan gemm_plan(int M, int N, int K) {
  GemmPlan pl{1, 1};
  if (M > 256 && g_gemm_variant == 0 && g_gemm_splits == 0) return prefill_plan(M, N, K);
  if (M <= 64) {
    pl.tile = 4;
  } else {
    const double c1 = tile_cost(M, N, 256, 160, 1.0);
    const double c2 = tile_cost(M, N, 128, 128, 1.3);
    const double c3 = tile_cost(M, N, 256, 256, 0.9);
    pl.tile = (c3 < c1 && c3 < c2) ? 3 : (c2 < c1 ? 2 : 1);
  }
  if (g_gemm_variant > 0) pl.tile = g_gemm_variant;
  const int bm = kTiles[pl.tile].bm, bn = kTiles[pl.tile].bn;
  const long tiles = (long)((M + bm - 1) / bm) * ((N + bn - 1) / bn);
  const int kt = K / kBK;
  if (tiles < 100) {
    int s = (int)((200 + tiles / 2) / tiles);
    const int cap = kt / 8 > 0 ? kt / 8 : 1;  // at least 8 k-tiles per split
    if (s > cap) s = cap;
    if (s > 32) s = 32;
    if (s < 1) s = 1;
    pl.splits = s;
  }
  if (g_gemm_splits > 0) pl.splits = g_gemm_splits < kt ? g_gemm_splits : kt;
  // decode-sized launch that would need a second, mostly empty round: re-plan by bytes per compute unit
  if (M <= 256 && tiles * pl.splits > 256 && g_gemm_variant == 0 && g_gemm_splits == 0) return decode_plan(M, N, K);
  return pl;
}

void gemm_tile_shape(int tile, int* tile_rows, int* tile_cols) {
  *tile_rows = kTiles[tile].bm;
  *tile_cols = kTiles[tile].bn;
}

void gemm_describe(int M, int N, int K, int* tile_rows, int* tile_cols, int* splits, int* cut_cols) {
  const GemmPlan pl = gemm_plan(M, N, K);
  *tile_rows = kTiles[pl.tile].bm;
  *tile_cols = kTiles[pl.tile].bn;
  *splits = pl.splits;
  *cut_cols = pl.cut_cols;
}

int gemm_splits(int M, int N, int K) {
  if (M <= 0 || N <= 0 || K < kBK || K % kBK != 0) return 1;
  return gemm_plan(M, N, K).splits;
}

// Bytes of split-K partials a launch with exactly M rows needs.
// Splits stay within one round of 256 workgroups, so a product of more than 128 of the largest tiles has none; known without
// a plan, which matters to whoever sizes a workspace for all row counts up to some thousand.
static bool never_split(int M, int N) {
  constexpr int kLargest = 256 * 256;
  constexpr auto fits = [] {
    for (const Tile& t : kTiles)
      if (t.bm * t.bn > kLargest) return false;
    return true;
  };
  static_assert(fits(), "tiles");
  return M > 256 && (double)M * N > 128.0 * kLargest && g_gemm_variant == 0 && g_gemm_splits == 0;
}

size_t layer_partial_bytes(int M, int N, int K) {
  if (never_split(M, N)) return 0;
  const GemmPlan pl = layer_plan(M, N, K, ~(size_t)0);
  return pl.splits > 1 ? (size_t)pl.splits * M * N * sizeof(float) : 0;
}

size_t gemm_workspace_bytes(int M, int N, int K) {
  if (M <= 0 || N <= 0 || K < kBK || K % kBK != 0 || never_split(M, N)) return 0;
  const GemmPlan pl = gemm_plan(M, N, K);
  return pl.splits > 1 ? (size_t)pl.splits * M * N * sizeof(float) : 0;
}

hipError_t launch_gemm(const void* X, const void* W, int M, int N, int K, const Epilogue& ep,
                       hipStream_t stream, void* workspace, const SkinnyFused* fused, bool* fused_done) {
  if (M <= 0 || N <= 0 || K < kBK || K % kBK != 0) return M <= 0 || N <= 0 ? hipSuccess : hipErrorInvalidValue;
  return launch_gemm(X, W, M, N, K, ep, gemm_plan(M, N, K), stream, workspace, fused, fused_done);
}

hipError_t launch_gemm(const void* X, const void* W, int M, int N, int K, const Epilogue& ep, GemmPlan pl,
                       hipStream_t stream, void* workspace, const SkinnyFused* fused, bool* fused_done) {
  if (fused_done) *fused_done = false;
  if (M <= 0 || N <= 0) return hipSuccess;
  if (K < kBK || K % kBK != 0 || N % 8 != 0 || ep.seg_cols <= 0 || ep.seg_cols % 8 != 0 || ep.seg_cols_kv < 0 ||
      ep.seg_cols_kv % 8 != 0)
    return hipErrorInvalidValue;
  if (ep.residual && ep.seg_cols != N) return hipErrorInvalidValue;
  if (ep.x_ld != 0 && (ep.x_ld < K || ep.x_ld % 8 != 0)) return hipErrorInvalidValue;
  if (ep.out_ld != 0 && (ep.out_ld < N || ep.out_ld % 8 != 0 || ep.seg_cols != N)) return hipErrorInvalidValue;
  // operand offsets inside the kernel are 32-bit element counts
  if ((unsigned long long)M * (ep.x_ld > 0 ? ep.x_ld : K) >= (1ull << 32) || (unsigned long long)N * K >= (1ull << 32))
    return hipErrorInvalidValue;
  GemmParams p;
  p.X = (const uint16_t*)X;
  p.W = (const uint16_t*)W;
  p.bias = (const uint16_t*)ep.bias;
  p.residual = (const uint16_t*)ep.residual;
  for (int i = 0; i < 3; ++i) p.out[i] = (uint16_t*)ep.out[i];
  p.seg_cols = ep.seg_cols;
  p.seg_cols_kv = ep.seg_cols_kv > 0 ? ep.seg_cols_kv : ep.seg_cols;
  p.ldx = ep.x_ld > 0 ? ep.x_ld : K;
  p.ld_out = ep.out_ld > 0 ? ep.out_ld : ep.seg_cols;
  p.ld_res = N;
  p.n_base = 0;
  p.spread = 0;
  p.M = M; p.N = N; p.K = K;
  p.relu = ep.relu;
  p.tiles_m = p.tiles_n = 0;
  p.splits = 1;
  p.partial = nullptr;
  p.ctx_lens = nullptr; p.block_tables = nullptr; p.max_blocks = 0;
  p.k_cache = nullptr; p.v_cache = nullptr; p.n_heads = 0; p.n_kv_heads = 0; p.head_dim = 0;
#ifdef DS_DEV_STAMPS
  p.dbg = g_gemm_dbg;
#endif
  if (pl.splits > 1 && workspace == nullptr) pl.splits = 1;  // no room for partials: slower, still right
  if (pl.splits > 1 && ep.out_ld != 0) return hipErrorInvalidValue;  // the reduce pass writes dense rows
  const bool want_kv = fused && fused->kind == SkinnyFused::kKvAppend && ep.seg_cols == N && !ep.relu &&
                       !ep.residual && N == (fused->n_heads + 2 * fused->n_kv_heads) * fused->head_dim &&
                       fused->head_dim % 8 == 0;
  if (pl.splits > 1) {
    p.partial = (float*)workspace;
  } else if (want_kv && kTiles[pl.tile].kv && (pl.cut_cols == 0 || kTiles[pl.tail_tile].kv)) {
    // unsplit: the tile kernels' own epilogue scatters K and V into the cache
    p.ctx_lens = fused->ctx_lens; p.block_tables = fused->block_tables; p.max_blocks = fused->max_blocks;
    p.k_cache = (uint16_t*)fused->k_cache; p.v_cache = (uint16_t*)fused->v_cache;
    p.n_heads = fused->n_heads; p.n_kv_heads = fused->n_kv_heads; p.head_dim = fused->head_dim;
    if (fused_done) *fused_done = true;
  }
  hipError_t e;
  if (pl.cut_cols > 0 && pl.splits == 1) {
    // Leading columns on the large tile in whole rounds of 256 workgroups, the rest on a smaller tile: two
    // launches over disjoint column ranges [0, cut) and [cut, N) of the same product (same operands, bias,
    // residual and output segments; only the column range differs).
    GemmParams a = p, b = p;
    a.N = pl.cut_cols;
    b.n_base = pl.cut_cols;
    e = launch_tile(pl.tile, a, 1, pl.in_layer, stream);
    if (e != hipSuccess) return e;
    return launch_tile(pl.tail_tile, b, 1, pl.in_layer, stream);
  }
  e = launch_tile(pl.tile, p, pl.splits, pl.in_layer, stream);
  if (e != hipSuccess) return e;
  if (pl.splits > 1) e = launch_splitk_reduce(p.partial, pl.splits, M, N, ep, fused, fused_done, stream);
  return e;
}

}  // namespace ds
