// The bf16 tiles of the GEMM and the launches of both operand types.
#include "gemm_tiles.h"

namespace wam {
namespace {
// 288x128: 4 wavefronts of 288x32, one per SIMD, each with the accumulators of nine MFMA tiles
// (512 registers per lane): per slice it reads 10 fragments for 9 MFMAs and loads 53 KB for
// half as many again as 192x128 tiles' products.  It pays most where it makes one round of what
// is otherwise one and a part: 544 x 13824 at K = 5120, cold weights, 216 tiles 86.8 us against
// 119 in 256x256 tiles, the next best (a library product 82.6), 1560 x 5120 92.6 against 112 in
// 192x256 ones; in two rounds 1088 x 15360 170 against 182 in 192x128 ones.  Where 128x256 tiles
// fill their rounds they are faster (3152 x 5120: 155 against 182 us).
// 128x128 twice: 8 wavefronts with four stages hide a slice's latency alone on a CU, two
// workgroups of 4 wavefronts with two stages each other's where a short K and more tiles than
// CUs meet (FP8, 5304 x 1536 at K = 1536: 25.3 us against 28.6 in the next best tile).
struct Bf16Tiles {
  using C64 = Cfg<64, 64, 64, 4, 2, 2, 2, 2, 1, 1>;
  using C128 = Cfg<128, 128, 64, 4, 4, 2, 2, 2, 1, 1>;
  using C128x2 = Cfg<128, 128, 64, 2, 2, 2, 2>;
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
hipError_t launch_any(const GemmArgs& gin, const GemmGroup* gg, hipStream_t s) {
  GemmArgs g = gin;
  if (g.a_rows <= 0) { g.a_rows = g.M; g.a_bs = 0; }
  if (g.o_rows <= 0) { g.o_rows = g.M; g.o_bs = 0; }
  if (g.gate_rows <= 0) { g.gate_rows = g.M; g.gate_stride = 0; }
  const GemmPlan p = plan_gemm(g.M, g.N, g.K, g.fp8, g.epi == WAM_EPI_GELU_MX8, gg ? gg->n : 1, cu_count());
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
