// The panel kernel's tiles (15-17 of the block kernel's list), and the row sums that its fused norm reads.
#include "gemm_panel.h"

namespace sf {
namespace {

// Row sums of squares for the fused norm, [split_k][M]: eight lanes per row, lane c adds the 16-byte chunks c of the slices in
// order, with the instruction and in the order of the kernels that square while they multiply: the same bits.  A launch of
// its own takes 4 us (1280 x 4096: the rows come from L2) where v_dot2 among the panel kernel's products costs 20 to 30: it
// holds up the matrix instructions.
__global__ __launch_bounds__(256) void row_squares_kernel(const bf16_t *__restrict__ A, int M, int K, int kt_per_split,
                                                          float *__restrict__ ssq) {
#ifdef __HIP_DEVICE_COMPILE__
  constexpr int AHEAD = 16;
  const int row = blockIdx.x * 32 + (threadIdx.x >> 3), c = threadIdx.x & 7, ks = blockIdx.y;
  const int kt0 = ks * kt_per_split, kt1 = min(K / BK, kt0 + kt_per_split);
  const uint4 *p = reinterpret_cast<const uint4 *>(A + (size_t)min(row, M - 1) * K) + c;
  float t = 0.f;
  for (int i = kt0; i < kt1; i += AHEAD) {
    uint4 v[AHEAD];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) v[u] = p[(size_t)min(i + u, kt1 - 1) * 8];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u)
      if (i + u < kt1) {
        const uint32_t w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
        for (int q = 0; q < 4; ++q)
          t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w[q]), __builtin_bit_cast(bf16x2, w[q]), t, false);
      }
  }
  t += __shfl_xor(t, 1);
  t += __shfl_xor(t, 2);
  t += __shfl_xor(t, 4);
  if (c == 0 && row < M) ssq[(size_t)ks * M + row] = t;
#endif
}

}  // namespace

hipError_t launch_row_squares(const GemmArgs &a, int split_k, int kt_per_split, float *ssq, hipStream_t s) {
  row_squares_kernel<<<dim3((a.M + 31) / 32, split_k), 256, 0, s>>>((const bf16_t *)a.x, a.M, a.K, kt_per_split, ssq);
  return hipGetLastError();
}

//   id  rows x columns  waves      a wave's tiles
//   15  320 x 256       2 x 2      10 x 8
//   16  256 x 256       2 x 2       8 x 8
//   17  192 x 256       2 x 2       6 x 8
hipError_t dispatch_panel(int tile, const GemmArgs &a, hipStream_t s, int split) {
  switch (tile) {
    case 15: return run_panel<2, 2, 10, 8>(a, s, split);
    case 16: return run_panel<2, 2, 8, 8>(a, s, split);
    case 17: return run_panel<2, 2, 6, 8>(a, s, split);
    default: return hipErrorInvalidValue;
  }
}

hipError_t prepare_panel() {
  hipError_t err = ensure_panel_lds<2, 2, 10, 8>();
  if (err == hipSuccess) err = ensure_panel_lds<2, 2, 8, 8>();
  if (err == hipSuccess) err = ensure_panel_lds<2, 2, 6, 8>();
  return err;
}

}  // namespace sf
