// Instances of the product kernel for the forward products (both operands k-contiguous).
#include "gemm_tile.h"

namespace ls {

hipError_t gemm_nt(const GemmArgs& a, GemmTile t, hipStream_t s) {
  switch (a.epi) {
    case EPI_BF16:
      switch (t) {
        case TILE_256: return launch<true, true, EPI_BF16, 256, 256>(a, s);
        case TILE_256x192: return launch<true, true, EPI_BF16, 256, 192>(a, s);
        case TILE_128: return launch_small<true, true, EPI_BF16, 2>(a, s);
        case TILE_128_DEEP: return launch_small<true, true, EPI_BF16, 4>(a, s);
        default: return hipErrorInvalidValue;
      }
    case EPI_RESID:
      switch (t) {
        case TILE_256: return launch<true, true, EPI_RESID, 256, 256>(a, s);
        case TILE_256x192: return launch<true, true, EPI_RESID, 256, 192>(a, s);
        case TILE_128: return launch_small<true, true, EPI_RESID, 2>(a, s);
        case TILE_128_DEEP: return launch_small<true, true, EPI_RESID, 4>(a, s);
        default: return hipErrorInvalidValue;
      }
    case EPI_ROPE:
      if (a.head_dim == 64) {
        switch (t) {
          case TILE_256: return launch<true, true, EPI_ROPE64, 256, 256>(a, s);
          case TILE_128: return launch_small<true, true, EPI_ROPE64, 2>(a, s);
          case TILE_128_DEEP: return launch_small<true, true, EPI_ROPE64, 4>(a, s);
          default: return hipErrorInvalidValue;
        }
      }
      switch (t) {
        case TILE_256: return launch<true, true, EPI_ROPE, 256, 256>(a, s);
        case TILE_128: return launch_small<true, true, EPI_ROPE, 2>(a, s);
        case TILE_128_DEEP: return launch_small<true, true, EPI_ROPE, 4>(a, s);
        default: return hipErrorInvalidValue;
      }
    case EPI_GLU_FWD:
      switch (t) {
        case TILE_256: return launch<true, true, EPI_GLU_FWD, 256, 256>(a, s);
        case TILE_128: return launch_small<true, true, EPI_GLU_FWD, 2>(a, s);
        case TILE_128_DEEP: return launch_small<true, true, EPI_GLU_FWD, 4>(a, s);
        default: return hipErrorInvalidValue;
      }
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ls
