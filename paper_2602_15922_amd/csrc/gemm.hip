// The bf16 tiles of the GEMM and the choice of tiles for both operand types.
#include "gemm_tiles.h"

namespace wam {
namespace {
// 288x128: 4 wavefronts of 288x32, one per SIMD, each with the accumulators of nine MFMA tiles
// (512 registers per lane): per slice it reads 10 fragments for 9 MFMAs and loads 53 KB for
// half as many again as 192x128 tiles' products.  It pays where it makes one round of what is
// otherwise one and a part: 544 x 13824 at K = 5120, cold weights, 216 tiles 86.8 us
// against 102 in 192x128 tiles (a library product 82.6); a block of 544 rows at d = 5120 600 ->
// 577 us, the cache update of 1560 rows 1640 -> 1579.  Where more rounds run,
// 128x256 tiles are faster (3152 x 5120: 150 against 169 us).
struct Bf16Tiles {
  using C64 = Cfg<64, 64, 64, 4, 2, 2, 2, 2, 1, 1>;
  using C128 = Cfg<128, 128, 64, 4, 4, 2, 2, 2, 1, 1>;
  using C192n = Cfg<192, 128, 64, 3, 2, 4, 2, 2, 2, 1>;
  using C288 = Cfg<288, 128, 64, 3, 1, 4, 1, 2, 4, 3>;
  using C128w = Cfg<128, 256, 64, 3, 2, 4, 2, 2, 2, 2>;
  using C192 = Cfg<192, 256, 64, 2, 2, 4, 2>;
  using C256 = Cfg<256, 256, 64, 2, 2, 4, 2>;
};

hipError_t launch_gemm_bf16(const GemmArgs& g, const GemmPlan& p, const GemmGroup* gg, hipStream_t s) {
  if (gg) return launch_group_plan<Bf16Tiles>(g, p, *gg, s);
  switch (g.epi) {
    case WAM_EPI_BF16: return launch_plan<Bf16Tiles, WAM_EPI_BF16>(g, p, s);
    case WAM_EPI_GELU_BF16: return launch_plan<Bf16Tiles, WAM_EPI_GELU_BF16>(g, p, s);
    case WAM_EPI_RESID_F32: return launch_plan<Bf16Tiles, WAM_EPI_RESID_F32>(g, p, s);
    case WAM_EPI_F32: return launch_plan<Bf16Tiles, WAM_EPI_F32>(g, p, s);
    case WAM_EPI_ROPE: return launch_plan<Bf16Tiles, WAM_EPI_ROPE>(g, p, s);
    default: return hipErrorInvalidValue;
  }
}
}  // namespace

// Compute units of the current device (queried once per device).
int cu_count() {
  static int cus[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cus[dev] == 0) {
    int n = 0;
    cus[dev] = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0 ? n : 256;
  }
  return cus[dev];
}

namespace {
// What a tile costs (us), from launches with cold weights (each its own W, as in a model's
// step) over M = 32 ... 3152, N = 16 ... 15360, K = 512 ... 13824: `slice` per 128-byte slice
// of K for a workgroup alone on its CU, `fixed` for the launch, the prologue and the
// epilogue.  FP8 and bf16 slices cost about the same: both are held by the loads into LDS
// (64 bytes per cycle and CU) and their latency.
struct TileCost {
  int bm, bn;
  double slice, fixed;
  int per_cu;
};
constexpr TileCost COST[NTILES] = {
    {64, 64, 0.25, 5.0, 2},   {128, 128, 0.48, 6.5, 1}, {192, 128, 0.73, 7.0, 1}, {288, 128, 0.95, 9.0, 1},
    {128, 256, 0.85, 7.0, 1}, {192, 256, 1.30, 8.0, 1}, {256, 256, 1.42, 9.0, 1},
};
// two 64x64 workgroups on a CU share it: a slice of each takes twice as long
constexpr double SHARED = 2.0;

GemmPlan plan_gemm(const GemmArgs& g, int ng) {
  const long cus = cu_count();
  const int slices = (g.K * (g.fp8 ? 1 : 2) + 127) / 128;
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
    if (g.epi == WAM_EPI_GELU_MX8 && (t == TILE_64x64 || t == TILE_192x128)) continue;
    if (g.fp8 && t == TILE_288x128) continue;  // bf16 only
    const long tiles = ng * up(g.M, c.bm) * up(g.N, c.bn), slots = cus * c.per_cu & ~7L;
    const double sl = c.per_cu > 1 && tiles > cus ? c.slice * SHARED : c.slice;
    GemmPlan p;
    p.tile = t;
    const double cost = up(tiles, slots) * (slices * sl + c.fixed);
    if (t == 0 || least == 0.0 || cost < least) {
      least = cost;
      best = p;
    }
  }
  // Two column ranges, a taller one first and a shorter one (gemm_nt2: dispatch slots in
  // order, so the first workgroup is always among the busiest): n tiles of a height cost n
  // times its round.  At M = 3152, K = 5120, bf16: QKV (60 column tiles) 19 columns of 256-row
  // tiles and 41 of 128-row ones, 416 us measured against 441 for 192 rows alone; FFN1 (54)
  // 39 columns of 256-row tiles and 15 of 192-row ones, 369 against 383 us for 256 alone.  A
  // split must beat one height by 3%; among equal splits, the least total work.
  if (ng == 1 && up(g.M, 128) * up(g.N, 256) >= cus) {
    const int tile[3] = {TILE_128x256, TILE_192x256, TILE_256x256};
    const long ncol = up(g.N, 256);
    double best2 = 0.0, work2 = 0.0;
    for (int a = 1; a < 3; ++a)
      for (int b = 0; b < a; ++b) {
        const TileCost &ca = COST[tile[a]], &cb = COST[tile[b]];
        const double ra = slices * ca.slice + ca.fixed, rb = slices * cb.slice + cb.fixed;
        for (long c1 = 1; c1 < ncol; ++c1) {
          const long t1 = up(g.M, ca.bm) * c1, t2 = up(g.M, cb.bm) * (ncol - c1);
          const long n1 = up(t1, cus), n2 = up(t1 + t2, cus) - n1;
          const double c = ra * n1 + rb * n2, work = ra * t1 + rb * t2;
          if (c < 0.97 * least && (best.two < 0 || c < best2 || (c == best2 && work < work2))) {
            best2 = c; work2 = work;
            best = GemmPlan{};
            best.tile = tile[a]; best.two = tile[b]; best.c1 = (int)c1;
          }
        }
      }
  }
  return best;
}

hipError_t launch_any(const GemmArgs& gin, const GemmGroup* gg, hipStream_t s) {
  GemmArgs g = gin;
  if (g.a_rows <= 0) { g.a_rows = g.M; g.a_bs = 0; }
  if (g.o_rows <= 0) { g.o_rows = g.M; g.o_bs = 0; }
  if (g.gate_rows <= 0) { g.gate_rows = g.M; g.gate_stride = 0; }
  const GemmPlan p = plan_gemm(g, gg ? gg->n : 1);
  return g.fp8 ? launch_gemm_fp8(g, p, gg, s) : launch_gemm_bf16(g, p, gg, s);
}
}  // namespace

hipError_t launch_gemm(const GemmArgs& g, hipStream_t s) { return launch_any(g, nullptr, s); }

hipError_t launch_gemm_group(const GemmArgs& g, const GemmGroup& gg, hipStream_t s) {
  if (gg.n < 1 || gg.n > WAM_GEMM_GROUP_MAX || g.epi != WAM_EPI_BF16) return hipErrorInvalidValue;
  if (gg.n > 1) return launch_any(g, &gg, s);
  GemmArgs one = g;  // a group of one takes every plan
  one.W = gg.W[0];
  one.bias = gg.bias[0];
  one.out = gg.out[0];
  one.w_scale = gg.w_scale[0];
  return launch_any(one, nullptr, s);
}

}  // namespace wam
