// Instances of the product kernel for the input-gradient products (k-strided B).
#include "gemm_tile.h"

namespace ls {

hipError_t gemm_nn(const GemmArgs& a, GemmTile t, hipStream_t s) {
  switch (a.epi) {
    case EPI_BF16:
      switch (t) {
        case TILE_256: return launch<true, false, EPI_BF16, 256, 256>(a, s);
        case TILE_256x192: return launch<true, false, EPI_BF16, 256, 192>(a, s);
        default: return launch_narrow<true, false, EPI_BF16>(a, t, s);
      }
    case EPI_GLU_BWD:
      switch (t) {
        case TILE_256: return launch<true, false, EPI_GLU_BWD, 256, 256>(a, s);
        default: return launch_narrow<true, false, EPI_GLU_BWD>(a, t, s);
      }
    case EPI_PART: return t == TILE_256 ? launch<true, false, EPI_PART, 256, 256>(a, s) : hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ls
