// The FP8 (E4M3) tiles of the GEMM: slices of 128 bytes per row, as the bf16 tiles' slices,
// so the same tile shapes and rings; half the matrix-core time per byte.  Measured at K = 5120
// (40 slices) with cold weights, M x N: 544 x 5120 38.8 us in 128x128 tiles of 4 wavefronts
// and 2 stages, 26.3 in 8 wavefronts and 4 stages.
#include "gemm_tiles.h"

namespace wam {
namespace {
// (The 4x2 wave grid gives a wave of a 128x128 tile 64 columns, one block of the block-scaled
// output.)
struct Fp8Tiles {
  using C64 = Cfg<64, 64, 128, 4, 2, 2, 2, 1, 2, 2>;
  using C128 = Cfg<128, 128, 128, 4, 4, 2, 2, 1, 2, 2>;
  using C128x2 = Cfg<128, 128, 128, 2, 2, 2, 2, 1>;
  using C192n = Cfg<192, 128, 128, 3, 2, 4, 2, 1, 3, 2>;
  using C288 = void;  // for wide products such as FFN1, whose block-scaled output its 32-column waves cannot write
  using C128w = Cfg<128, 256, 128, 3, 2, 4, 2, 1, 3, 3>;
  using C192 = Cfg<192, 256, 128, 2, 2, 4, 2, 1>;
  using C256 = Cfg<256, 256, 128, 2, 2, 4, 2, 1>;
};
}  // namespace

hipError_t launch_gemm_fp8(const GemmArgs& g, const GemmPlan& p, const GemmGroup* gg, hipStream_t s) {
  if (gg) return launch_group_plan<Fp8Tiles>(g, p, *gg, s);
  switch (g.epi) {
    case WAM_EPI_BF16: return launch_plan<Fp8Tiles, WAM_EPI_BF16>(g, p, s);
    case WAM_EPI_GELU_BF16: return launch_plan<Fp8Tiles, WAM_EPI_GELU_BF16>(g, p, s);
    case WAM_EPI_RESID_F32: return launch_plan<Fp8Tiles, WAM_EPI_RESID_F32>(g, p, s);
    case WAM_EPI_F32: return launch_plan<Fp8Tiles, WAM_EPI_F32>(g, p, s);
    case WAM_EPI_GELU_MX8: return launch_plan<Fp8Tiles, WAM_EPI_GELU_MX8>(g, p, s);
    case WAM_EPI_MXA | WAM_EPI_BF16: return launch_plan<Fp8Tiles, WAM_EPI_MXA | WAM_EPI_BF16>(g, p, s);
    case WAM_EPI_MXA | WAM_EPI_RESID_F32: return launch_plan<Fp8Tiles, WAM_EPI_MXA | WAM_EPI_RESID_F32>(g, p, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace wam
