// Tile configurations of the bf16 linear layers: eight waves, 192-320 rows x 256 columns.
#include "gemm_ring.h"

namespace sf {

hipError_t dispatch_tall(int tile, const GemmArgs &a, hipStream_t s, int split) {
  switch (tile) {
    case 11: return run_ring<10, 1, 2, 1, 8, 2, 0>(a, s, split);
    case 12: return run_ring<8, 1, 2, 1, 8, 2, 0>(a, s, split);
    case 13: return run_ring<7, 1, 2, 1, 8>(a, s, split);
    case 14: return run_ring<6, 1, 3, 1, 8>(a, s, split);
    default: return hipErrorInvalidValue;
  }
}

hipError_t prepare_tall() {
  hipError_t err = ensure_lds<10, 1, 2, 1, 8, 2, 0>();
  if (err == hipSuccess) err = ensure_lds<8, 1, 2, 1, 8, 2, 0>();
  if (err == hipSuccess) err = ensure_lds<7, 1, 2, 1, 8>();
  if (err == hipSuccess) err = ensure_lds<6, 1, 3, 1, 8>();
  return err;
}

}  // namespace sf
