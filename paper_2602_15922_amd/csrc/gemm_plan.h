// How a GEMM launch deals its product to tiles: the choice alone, host code with no HIP in it.
#pragma once

namespace wam {

// The tiles a product can run in (rows x columns; gemm_tiles.h's users instantiate each for
// their operand type).  128x128: 8 wavefronts and four stages, alone on a CU; 128x128_2: 4
// wavefronts and two stages, two workgroups per CU.
enum GemmTile {
  TILE_64x64, TILE_128x128, TILE_192x128, TILE_288x128, TILE_128x256, TILE_192x256, TILE_256x256, TILE_128x128_2, NTILES
};
struct GemmPlan {
  int tile = TILE_128x256;
  int two = -1, c1 = 0;  // two column ranges: c1 columns of `tile`, the rest in tile `two`
};

// What a tile costs (us) per 128-byte slice of K: `alone` where a tile that shares a CU has no
// neighbour (tiles <= CUs), `one` in a launch of one round, `many` in a round of several;
// `fixed`: the prologue and the epilogue of a round and its share of the launch.  Fitted to
// launches with cold weights (each its own W, as in a model's step): every tile and pair of
// column ranges that came near the best one, timed in turn, for the projections of d = 512,
// 1536, 3072 and 5120, bf16 and FP8, over 75 row counts from 17 to 6304 (3040 products).  FP8
// and bf16 slices cost about the same: both are held by the loads into LDS (64 bytes per cycle
// and CU) and their latency.  The choice is within 0.3% of the fastest measured plan on
// average, past 3% for 1 product in 25.
struct TileCost {
  int bm, bn, per_cu;
  double alone, one, many, fixed;
};
constexpr TileCost COST[NTILES] = {
    {64, 64, 2, 0.265, 0.470, 0.340, 4.5},    {128, 128, 1, 0.507, 0.507, 0.466, 6.4},
    {192, 128, 1, 0.627, 0.627, 0.744, 7.5},  {288, 128, 1, 0.850, 0.850, 0.862, 24.7},
    {128, 256, 1, 0.860, 0.860, 0.800, 8.7},  {192, 256, 1, 1.150, 1.150, 1.286, 14.0},
    {256, 256, 1, 1.200, 1.200, 1.373, 19.0}, {128, 128, 2, 0.720, 1.050, 1.000, 6.3},
};

// ng products of M x N with K elements of 1 (FP8) or 2 bytes in one launch on `cus` compute
// units; mx8_out: the output is written block-scaled.
inline GemmPlan plan_gemm(int M, int N, int K, bool fp8, bool mx8_out, int ng, long cus) {
  const int slices = (int)(((long)K * (fp8 ? 1 : 2) + 127) / 128);
  auto up = [](long a, long b) { return (a + b - 1) / b; };
  // Every tile over all columns: a launch costs its rounds of resident workgroups.  K is never
  // split, whatever a tile leaves idle: every tile sums an output's products in the same order
  // (ascending K, one MFMA chain), so a row's bits depend neither on the tile nor on how many
  // rows the call has.
  GemmPlan best;
  double least = 0.0;
  for (int t = 0; t < NTILES; ++t) {
    const TileCost& c = COST[t];
    // the block-scaled output needs a wave's columns to be one 64-column block
    if (mx8_out && (t == TILE_64x64 || t == TILE_192x128)) continue;
    if (fp8 && t == TILE_288x128) continue;  // bf16 only
    const long tiles = ng * up(M, c.bm) * up(N, c.bn), rounds = up(tiles, cus * c.per_cu);
    const double slice = rounds > 1 ? c.many : tiles <= cus ? c.alone : c.one;
    const double cost = rounds * (slices * slice + c.fixed);
    if (t == 0 || least == 0.0 || cost < least) {
      least = cost;
      best = GemmPlan{};
      best.tile = t;
    }
  }
  // Two column ranges, a taller one first and a shorter one (gemm_nt2: dispatch slots in
  // order, so the first workgroup is always among the busiest): n tiles of a height cost n
  // times its round.  At M = 3152, K = 5120, bf16, cold weights: QKV (60 column tiles) 19 columns
  // of 256-row tiles and 41 of 128-row ones, 433 us against 446 for 128-row tiles alone; FFN1 (54) 39 columns of 256-row tiles
  // and 15 of 192-row ones, 395 against 405 us for 256 alone (FP8 233 against 239).  A pair must beat one tile by 1%; among equal pairs, the
  // least time in the slices.
  if (ng == 1 && up(M, 128) * up(N, 256) >= cus) {
    const int tile[3] = {TILE_128x256, TILE_192x256, TILE_256x256};
    const long ncol = up(N, 256);
    double best2 = 0.0, work2 = 0.0;
    for (int a = 1; a < 3; ++a)
      for (int b = 0; b < a; ++b) {
        const TileCost &ca = COST[tile[a]], &cb = COST[tile[b]];
        const double ra = slices * ca.many + ca.fixed, rb = slices * cb.many + cb.fixed;
        for (long c1 = 1; c1 < ncol; ++c1) {
          const long t1 = up(M, ca.bm) * c1, t2 = up(M, cb.bm) * (ncol - c1);
          const long n1 = up(t1, cus), n2 = up(t1 + t2, cus) - n1;
          const double c = ra * n1 + rb * n2, work = ca.many * t1 + cb.many * t2;
          if (c < 0.99 * least && (best.two < 0 || c < best2 || (c == best2 && work < work2))) {
            best2 = c;
            work2 = work;
            best.tile = tile[a];
            best.two = tile[b];
            best.c1 = (int)c1;
          }
        }
      }
  }
  return best;
}

}  // namespace wam
