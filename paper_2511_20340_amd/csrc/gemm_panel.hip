// The panel kernel's tiles, and the row sums that its fused norm reads.
#include "gemm_panel.h"

namespace sf {
namespace {

// Row sums of squares for the fused norm, [split_k][M]: eight lanes per row, lane c adds the 16-byte chunks c of the slices in
// order, with the instruction and in the order of the kernels that square while they multiply: the same bits.  A launch of
// its own takes 4 us (1280 x 4096: the rows come from L2) where v_dot2 among the panel kernel's products costs 20 to 30: it
// holds up the matrix instructions.
__global__ __launch_bounds__(64, 1) void row_squares_kernel(const bf16_t *__restrict__ A, int M, int K, int kt_per_split,
                                                          float *__restrict__ ssq) {
#ifdef __HIP_DEVICE_COMPILE__
  constexpr int AHEAD = 32;  // slices of a row requested at a time: all of K = 2048
  const int row = blockIdx.x * 8 + (threadIdx.x >> 3), c = threadIdx.x & 7, ks = blockIdx.y;
  const int kt0 = ks * kt_per_split, kt1 = min(K / BK, kt0 + kt_per_split);
  const uint4 *p = reinterpret_cast<const uint4 *>(A + (size_t)min(row, M - 1) * K) + c;
  float t = 0.f;
  uint4 v[2][AHEAD];
  auto request = [&](int h, int i) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) v[h][u] = p[(size_t)min(i + u, kt1 - 1) * 8];
  };
  auto add = [&](int h, int i) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < AHEAD; ++u)
      if (i + u < kt1) {
        const uint32_t w[4] = {v[h][u].x, v[h][u].y, v[h][u].z, v[h][u].w};
#pragma unroll
        for (int q = 0; q < 4; ++q)
          t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w[q]), __builtin_bit_cast(bf16x2, w[q]), t, false);
      }
  };
  request(0, kt0);
  for (int i = kt0; i < kt1; i += 2 * AHEAD) {
    if (i + AHEAD < kt1) request(1, i + AHEAD);
    add(0, i);
    if (i + AHEAD >= kt1) break;
    if (i + 2 * AHEAD < kt1) request(0, i + 2 * AHEAD);
    add(1, i + AHEAD);
  }
  t += __shfl_xor(t, 1);
  t += __shfl_xor(t, 2);
  t += __shfl_xor(t, 4);
  if (c == 0 && row < M) ssq[(size_t)ks * M + row] = t;
#endif
}

}  // namespace

hipError_t launch_row_squares(const GemmArgs &a, int split_k, int kt_per_split, float *ssq, hipStream_t s) {
  row_squares_kernel<<<dim3((a.M + 7) / 8, split_k), 64, 0, s>>>((const bf16_t *)a.x, a.M, a.K, kt_per_split, ssq);
  return hipGetLastError();
}

//   id  rows x columns  a wave's tiles  slices, workgroups per CU
//   15  320 x 256       10 x 8          2, 1
//   16  256 x 256        8 x 8          2, 1
//   17  192 x 256        6 x 8          2, 1
//   18  128 x 256        4 x 8          3, 1 (without the norm; with it: the block kernel)
//   26  128 x 128        4 x 4          4, 1
//   27  160 x 128        5 x 4          2, 2
//   28  160 x 128        5 x 4          4, 1
// Measured and left out: 320 x 192, 320 x 128, 160 x 256, 128 x 128 with two to a compute unit; loader waves that run the
// weights further ahead than the rows (no faster); reading later slices' weight lines ahead into L2 (no faster).
hipError_t dispatch_panel(int tile, const GemmArgs &a, hipStream_t s, int split) {
  switch (tile) {
    case 15: return run_panel<2, 2, 10, 8, 2>(a, s, split);
    case 16: return run_panel<2, 2, 8, 8, 2>(a, s, split);
    case 17: return run_panel<2, 2, 6, 8, 2>(a, s, split);
    default: return dispatch_panel_narrow(tile, a, s, split);
  }
}

hipError_t prepare_panel() {
  hipError_t err = ensure_panel_lds<2, 2, 10, 8, 2>();
  if (err == hipSuccess) err = ensure_panel_lds<2, 2, 8, 8, 2>();
  if (err == hipSuccess) err = ensure_panel_lds<2, 2, 6, 8, 2>();
  return err == hipSuccess ? prepare_panel_narrow() : err;
}

}  // namespace sf
