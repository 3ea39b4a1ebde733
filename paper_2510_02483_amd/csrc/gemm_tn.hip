// Instances of the product kernel for the weight-gradient products (both operands k-strided), fp32.
#include "gemm_tile.h"

namespace ls {

hipError_t gemm_tn(const GemmArgs& a, GemmTile t, hipStream_t s) {
  switch (a.epi) {
    case EPI_F32:
      switch (t) {
        case TILE_256: return launch<false, false, EPI_F32, 256, 256>(a, s);
        case TILE_256x192: return launch<false, false, EPI_F32, 256, 192>(a, s);
        case TILE_192x256: return launch<false, false, EPI_F32, 192, 256>(a, s);
        case TILE_192: return launch<false, false, EPI_F32, 192, 192>(a, s);
        default: return launch_narrow<false, false, EPI_F32>(a, t, s);
      }
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ls
