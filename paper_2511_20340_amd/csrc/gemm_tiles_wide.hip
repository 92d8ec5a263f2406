// Tile configurations of the bf16 linear layers: eight waves: 64-160 rows x 256 columns.
#include "gemm_ring.h"

namespace sf {

hipError_t dispatch_wide(int tile, const GemmArgs &a, hipStream_t s, int split) {
  switch (tile) {
    case 6: return run_ring<2, 1, 2, 1, 8, 1>(a, s, split);
    case 7: return run_ring<3, 1, 4, 1, 8, 1>(a, s, split);
    case 8: return run_ring<4, 1, 2, 1, 8, 1>(a, s, split);
    case 9: return run_ring<5, 1, 3, 1, 8>(a, s, split);
    case 10: return run_ring<5, 1, 2, 1, 8, 1>(a, s, split);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace sf
