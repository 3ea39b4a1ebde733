// Instances of the product kernel for the input-gradient products (k-strided B).
#include "gemm_tile.h"

namespace ls {

hipError_t gemm_nn(const GemmArgs& a, GemmTile t, hipStream_t s) {
  switch (a.epi) {
    case EPI_BF16:
      switch (t) {
        case TILE_256: return launch<true, false, EPI_BF16, 256, 256>(a, s);
        case TILE_256x192: return launch<true, false, EPI_BF16, 256, 192>(a, s);
        case TILE_128: return launch_small<true, false, EPI_BF16, 2>(a, s);
        case TILE_128_DEEP: return launch_small<true, false, EPI_BF16, 4>(a, s);
        default: return hipErrorInvalidValue;
      }
    case EPI_GLU_BWD:
      switch (t) {
        case TILE_256: return launch<true, false, EPI_GLU_BWD, 256, 256>(a, s);
        case TILE_128: return launch_small<true, false, EPI_GLU_BWD, 2>(a, s);
        case TILE_128_DEEP: return launch_small<true, false, EPI_GLU_BWD, 4>(a, s);
        default: return hipErrorInvalidValue;
      }
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ls
