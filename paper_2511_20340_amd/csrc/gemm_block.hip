// The block kernel's tile configurations.
#include "gemm_block.h"

namespace sf {

//   id  rows x columns  waves      LDS slices, workgroups per CU
//   18  128 x 256       2 x 4      3, 1 (only with the fused norm)
//   29  320 x 256       2 x 4      2, 1 (29-31: only with the fused norm, unsplit, where its row sums of squares have no
//   30  256 x 256       2 x 4      2, 1  memory to go through on their way to the panel kernel: 2048 x 8192 x 8192 and
//   31  192 x 256       2 x 4      2, 1  1280 x 28672 x 4096 take 228 and 272 us, 272 and 326 on tile 18, 203 and 238 there)
//   19  128 x  64       2 x 2      3, 2
//   20   64 x  64       2 x 2      4, 2
//   21  160 x  64       5 x 1      5, 1
//   22  160 x 128       5 x 2      4, 1
//   15-17, 18 without the norm, 26-28: the panel kernel's (gemm_panel.hip)
// K shared by groups of waves (layers whose K is split that often, see gemm_block_kernel):
//   23   64 x  64       2 x 2, 2 groups   4, 1
//   24   32 x  64       1 x 2, 4 groups   3, 1
//   25   32 x  64       1 x 2, 2 groups   3, 2
// Measured and left out, as these are within 0.5 % of all of them over the measured shapes: 256 x 128, 160 x 256 and
// 64 x 256 (eight waves), 160 x 128, 128 x 128, 96 x 128, 64 x 128 and 32 x 128 (four); 64 x 64 in 4 groups, 128 x 64 and
// 64 x 128 in 2, 32 x 128 in 4, 32 x 32 in 8.
hipError_t dispatch_block(int tile, const GemmArgs &a, hipStream_t s, int split) {
  switch (tile) {
    case 18: return a.fused_norm ? run_block<2, 4, 2, 2, 3, 1, true>(a, s, split) : dispatch_panel(tile, a, s, split);
    case 19: return run_block<2, 2, 2, 1, 3>(a, s, split);
    case 20: return run_block<2, 2, 1, 1, 4>(a, s, split);
    case 21: return run_block<5, 1, 1, 2, 5>(a, s, split);
    case 22: return run_block<5, 2, 1, 2, 4>(a, s, split);
    case 23: return run_block<2, 2, 1, 1, 4, 2>(a, s, split);
    case 24: return run_block<1, 2, 1, 1, 3, 4>(a, s, split);
    case 25: return run_block<1, 2, 1, 1, 3, 2>(a, s, split);
    case 29: return run_block<2, 4, 5, 2, 2, 1, true>(a, s, split);
    case 30: return run_block<2, 4, 4, 2, 2, 1, true>(a, s, split);
    case 31: return run_block<2, 4, 3, 2, 2, 1, true>(a, s, split);
    default: return dispatch_panel(tile, a, s, split);
  }
}

hipError_t prepare_block() {
  hipError_t err = prepare_panel();
  if (err == hipSuccess) err = ensure_block_lds<2, 4, 2, 2, 3, 1, true>();
  if (err == hipSuccess) err = ensure_block_lds<2, 4, 5, 2, 2, 1, true>();
  if (err == hipSuccess) err = ensure_block_lds<2, 4, 4, 2, 2, 1, true>();
  if (err == hipSuccess) err = ensure_block_lds<2, 4, 3, 2, 2, 1, true>();
  if (err == hipSuccess) err = ensure_block_lds<2, 2, 2, 1, 3>();
  if (err == hipSuccess) err = ensure_block_lds<5, 2, 1, 2, 4>();
  if (err == hipSuccess) err = ensure_block_lds<2, 2, 1, 1, 4>();
  if (err == hipSuccess) err = ensure_block_lds<5, 1, 1, 2, 5>();
  if (err == hipSuccess) err = ensure_block_lds<2, 2, 1, 1, 4, 2>();
  if (err == hipSuccess) err = ensure_block_lds<1, 2, 1, 1, 3, 4>();
  if (err == hipSuccess) err = ensure_block_lds<1, 2, 1, 1, 3, 2>();
  return err;
}

int block_groups(int tile) { return tile == 24 ? 4 : tile == 23 || tile == 25 ? 2 : 1; }

// Whole slices of K; 32-bit byte offsets into both operands; arg-max partials are kept per 128 columns at the finest, and
// 26-28 are built without them (heads of many rows choose 15-18); a tile with groups takes the layers whose K is split that
// often; with the norm the panel kernel's row sums of squares go through memory: norm_ws bytes of the workspace
// (gemm_norm_bytes; -1: no norm), or, split, beside the partial tiles.
bool block_takes(int tile, int M, int N, int K, int split, bool am, ptrdiff_t norm_ws) {
  if (tile < 15 || tile > 31 || (am && tile >= 19 && tile != 22)) return false;
  const int parts = make_plan(M, N, K, 32, 32, split).split_k;
  if (block_groups(tile) > 1 && parts != block_groups(tile)) return false;
  // 26-28: unsplit layers only (split ones gain up to 6 % from them)
  if (tile > 25 && parts > 1) return false;
  if (squares_before(tile) && norm_ws >= 0 && parts == 1 && !squares_fit(M, norm_ws)) return false;
  if (tile > 28 && norm_ws < 0) return false;
  const size_t limit = (size_t)1 << 32;
  return K % BK == 0 && (size_t)M * K * 2 < limit && (size_t)((N + 31) / 32) * K * 64 < limit;
}

}  // namespace sf
