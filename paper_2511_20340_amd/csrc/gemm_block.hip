// The block kernel's tile configurations.
#include "gemm_block.h"

namespace sf {

//   id  rows x columns  waves      LDS slices, workgroups per CU
//   15  320 x 256       2 x 4      2, 1
//   16  256 x 256       2 x 4      2, 1
//   17  192 x 256       2 x 4      2, 1
//   18  128 x 256       2 x 4      3, 1
//   19  128 x  64       2 x 2      3, 2
//   20   64 x  64       2 x 2      4, 2
//   21  160 x  64       5 x 1      5, 1
//   22  160 x 128       5 x 2      4, 1
// Measured and left out, as these eight are within 0.3 % of all sixteen over the measured shapes: 256 x 128, 160 x 256 and
// 64 x 256 (eight waves), 160 x 128, 128 x 128, 96 x 128, 64 x 128 and 32 x 128 (four).
hipError_t dispatch_block(int tile, const GemmArgs &a, hipStream_t s, int split) {
  switch (tile) {
    case 15: return run_block<2, 4, 5, 2, 2>(a, s, split);
    case 16: return run_block<2, 4, 4, 2, 2>(a, s, split);
    case 17: return run_block<2, 4, 3, 2, 2>(a, s, split);
    case 18: return run_block<2, 4, 2, 2, 3>(a, s, split);
    case 19: return run_block<2, 2, 2, 1, 3>(a, s, split);
    case 20: return run_block<2, 2, 1, 1, 4>(a, s, split);
    case 21: return run_block<5, 1, 1, 2, 5>(a, s, split);
    case 22: return run_block<5, 2, 1, 2, 4>(a, s, split);
    default: return hipErrorInvalidValue;
  }
}

hipError_t prepare_block() {
  hipError_t err = ensure_block_lds<2, 4, 5, 2, 2>();
  if (err == hipSuccess) err = ensure_block_lds<2, 4, 4, 2, 2>();
  if (err == hipSuccess) err = ensure_block_lds<2, 4, 3, 2, 2>();
  if (err == hipSuccess) err = ensure_block_lds<2, 4, 2, 2, 3>();
  if (err == hipSuccess) err = ensure_block_lds<2, 2, 2, 1, 3>();
  if (err == hipSuccess) err = ensure_block_lds<2, 2, 1, 1, 4>();
  if (err == hipSuccess) err = ensure_block_lds<5, 1, 1, 2, 5>();
  if (err == hipSuccess) err = ensure_block_lds<5, 2, 1, 2, 4>();
  return err;
}

// Whole slices of K; 32-bit byte offsets into both operands; arg-max partials are kept per 128 columns at the finest.
bool block_takes(int tile, int M, int N, int K, bool am) {
  if (tile < 15 || tile > 22 || (am && tile >= 19 && tile <= 21)) return false;
  const size_t limit = (size_t)1 << 32;
  return K % BK == 0 && (size_t)M * K * 2 < limit && (size_t)((N + 31) / 32) * K * 64 < limit;
}

}  // namespace sf
