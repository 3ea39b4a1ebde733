// Instances of the product kernel for the forward products (both operands k-contiguous).
#include "gemm_tile.h"

namespace ls {

hipError_t gemm_nt(const GemmArgs& a, GemmTile t, hipStream_t s) {
  switch (a.epi) {
    case EPI_BF16:
      switch (t) {
        case TILE_256: return launch<true, true, EPI_BF16, 256, 256>(a, s);
        case TILE_256x192: return launch<true, true, EPI_BF16, 256, 192>(a, s);
        default: return launch_narrow<true, true, EPI_BF16>(a, t, s);
      }
    case EPI_RESID:
      switch (t) {
        case TILE_256: return launch<true, true, EPI_RESID, 256, 256>(a, s);
        case TILE_256x192: return launch<true, true, EPI_RESID, 256, 192>(a, s);
        default: return launch_narrow<true, true, EPI_RESID>(a, t, s);
      }
    case EPI_ROPE:
      if (a.head_dim == 64) {
        switch (t) {
          case TILE_256: return launch<true, true, EPI_ROPE64, 256, 256>(a, s);
          default: return launch_narrow<true, true, EPI_ROPE64>(a, t, s);
        }
      }
      switch (t) {
        case TILE_256: return launch<true, true, EPI_ROPE, 256, 256>(a, s);
        default: return launch_narrow<true, true, EPI_ROPE>(a, t, s);
      }
    case EPI_GLU_FWD:
      switch (t) {
        case TILE_256: return launch<true, true, EPI_GLU_FWD, 256, 256>(a, s);
        default: return launch_narrow<true, true, EPI_GLU_FWD>(a, t, s);
      }
    case EPI_PART: return t == TILE_256 ? launch<true, true, EPI_PART, 256, 256>(a, s) : hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ls
