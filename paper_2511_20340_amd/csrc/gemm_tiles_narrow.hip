// Tile configurations of the bf16 linear layers: four waves: 32-160 rows x 128 columns.
#include "gemm_ring.h"

namespace sf {

hipError_t dispatch_narrow(int tile, const GemmArgs &a, hipStream_t s, int split) {
  switch (tile) {
    case 1: return run_ring<1, 1, 4, 4, 4>(a, s, split);
    case 2: return run_ring<2, 1, 4, 3, 4>(a, s, split);
    case 3: return run_ring<3, 1, 4, 2, 4, 1>(a, s, split);
    case 4: return run_ring<4, 1, 2, 2, 4, 1>(a, s, split);
    case 5: return run_ring<5, 1, 2, 2, 4, 1>(a, s, split);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace sf
