// What the kernels of the bf16 linear layers and their host code share: the epilogue's arguments, row input / output,
// the K partition.
#pragma once
#include "sf_internal.h"

namespace sf {

constexpr int BK = 64;
constexpr int LDK = 72;  // padded LDS row length in bf16 elements (144 B)
constexpr int XCDS = 8;

// Where a workgroup's finished accumulators go.
struct Epilogue {
  const bf16_t *bias;    // [N] or null
  const void *residual;  // [M][N] bf16, or float when res_f32; may alias y
  void *y;               // [M][N] bf16, or float when out_f32; null: not stored (arg-max partials only)
  bf16_t *y2;            // optional bf16 copy of y
  bf16_t *hooks;         // optional: bf16 copies of block row (r / hook_q, r % hook_q) into the groups of hook_mask
  float *am_val;         // optional [M][am_stride]: per row and column tile the largest value ...
  int32_t *am_idx;       // ... and its column
  int hook_mask, hook_q, hook_qmax, am_stride;
  int out_f32, res_f32, glu;
  int vec;               // every pointer above is 16-byte aligned and so are the rows (N % 8 == 0)
};

// W (4 or 8) consecutive elements as floats; vec: every pointer of the launch is 16-byte aligned
template <int W>
__device__ __forceinline__ void load_n(const bf16_t *p, float (&v)[W], int vec) {
  typedef uint32_t words __attribute__((ext_vector_type(W / 2)));
  if (vec) {
    const words w = *reinterpret_cast<const words *>(p);
#pragma unroll
    for (int i = 0; i < W / 2; ++i) { v[2 * i] = __uint_as_float(w[i] << 16); v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u); }
  } else {
    for (int i = 0; i < W; ++i) v[i] = bf2f(p[i]);
  }
}
template <int W>
__device__ __forceinline__ void load_n(const float *p, float (&v)[W], int vec) {
  if (vec) {
#pragma unroll
    for (int j = 0; j < W / 4; ++j) {
      const f32x4 q = *reinterpret_cast<const f32x4 *>(p + j * 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[j * 4 + i] = q[i];
    }
  } else {
    for (int i = 0; i < W; ++i) v[i] = p[i];
  }
}
// n: elements that exist behind p (W or more where vec)
template <int W>
__device__ __forceinline__ void store_n(bf16_t *p, const float (&v)[W], int vec, int n = W) {
  typedef uint32_t words __attribute__((ext_vector_type(W / 2)));
  if (vec) {
    words w;
#pragma unroll
    for (int i = 0; i < W / 2; ++i) w[i] = pack2bf(v[2 * i], v[2 * i + 1]);
    *reinterpret_cast<words *>(p) = w;
  } else {
    for (int i = 0; i < W; ++i)
      if (i < n) p[i] = f2bf(v[i]);
  }
}
template <int W>
__device__ __forceinline__ void store_n(float *p, const float (&v)[W], int vec, int n = W) {
  if (vec) {
#pragma unroll
    for (int j = 0; j < W / 4; ++j) *reinterpret_cast<f32x4 *>(p + j * 4) = f32x4{v[j * 4], v[j * 4 + 1], v[j * 4 + 2], v[j * 4 + 3]};
  } else {
    for (int i = 0; i < W; ++i)
      if (i < n) p[i] = v[i];
  }
}

// W finished columns of an output row: y, its bf16 copy, the hooked copies.  Only y, the logits of an LM head, can have
// rows that end within the W.
template <int W>
__device__ __forceinline__ void store_row(const Epilogue &e, int row, int col, int N, const float (&r)[W]) {
  const size_t o = (size_t)row * N + col;
  if (e.out_f32) store_n(reinterpret_cast<float *>(e.y) + o, r, e.vec, N - col);
  else store_n(reinterpret_cast<bf16_t *>(e.y) + o, r, e.vec, N - col);
  if (e.y2) store_n(e.y2 + o, r, e.vec);
  if (e.hooks) {
    const size_t hrow = ((size_t)(row / e.hook_q) * e.hook_qmax + row % e.hook_q) * 4;
#pragma unroll
    for (int g = 1; g < 4; ++g)
      if (e.hook_mask >> g & 1) store_n(e.hooks + (hrow + g) * N + col, r, e.vec);
  }
}

struct Plan {
  int tiles_m, tiles_n, split_k, kt_per_split;
  size_t partial_bytes;
};

// split_k workgroups share a tile's K range.  The partition depends on K and split only -- never on
// the tile configuration -- because it fixes the fp32 summation order of every output element.
inline Plan make_plan(int M, int N, int K, int BM, int BN, int split) {
  Plan p;
  p.tiles_m = (M + BM - 1) / BM;
  p.tiles_n = (N + BN - 1) / BN;
  const int KT = (K + BK - 1) / BK;
  const int tiles = p.tiles_m * p.tiles_n;
  const int s = split < 1 ? 1 : (split > KT ? KT : split);
  p.kt_per_split = (KT + s - 1) / s;
  p.split_k = (KT + p.kt_per_split - 1) / p.kt_per_split;
  p.partial_bytes = p.split_k > 1 ? (size_t)tiles * p.split_k * BM * BN * sizeof(float) : 0;
  return p;
}

// workspace: [row sums of squares of the fused norm][partial tiles]
inline bool plan_fits(const Plan &p, int BM, const void *ws, size_t ws_bytes) {
  if (p.split_k == 1) return true;
  const size_t ssq_bytes = (size_t)p.tiles_m * p.split_k * BM * sizeof(float);
  return ws && ws_bytes >= GEMM_SSQ_BYTES + p.partial_bytes && ssq_bytes <= GEMM_SSQ_BYTES;
}

// The rest of a row's epilogue for 8 finished sums: bias, residual, outputs
__device__ __forceinline__ void finish_row8(const Epilogue &e, int row, int col, int N, float (&r)[8]) {
  const size_t o = (size_t)row * N + col;
  if (e.bias) {
    float bv[8];
    load_n(e.bias + col, bv, e.vec);
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] += bv[i];
  }
  if (e.residual) {
    float res[8];
    if (e.res_f32) load_n(reinterpret_cast<const float *>(e.residual) + o, res, e.vec);
    else load_n(reinterpret_cast<const bf16_t *>(e.residual) + o, res, e.vec);
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] += res[i];
  }
  store_row(e, row, col, N, r);
}

inline Epilogue make_epilogue(const GemmArgs &a) {
  const uintptr_t all = (uintptr_t)a.bias | (uintptr_t)a.residual | (uintptr_t)a.y | (uintptr_t)a.y2 | (uintptr_t)a.hooks;
  return Epilogue{(const bf16_t *)a.bias, a.residual, a.y, (bf16_t *)a.y2, (bf16_t *)a.hooks, a.am_val, a.am_idx,
                  a.hook_mask, a.hook_q, a.hook_qmax, a.am_stride, a.out_f32, a.res_f32, a.glu, (all & 15) == 0 && a.N % 8 == 0};
}

// Weights of a layer with one M-tile are read once per launch; from this size on they leave the caches alone
// (non-temporal loads stream faster from HBM, and a model of such layers does not fit the memory-side cache from one
// step to the next anyway).  Ring kernel, 5 rows: 28672 x 4096 47 -> 41 us, 128256 x 4096 183 -> 160, 4096 x 14336 26.6 -> 24.0,
// 4096 x 4096 (34 MB) 13.1 -> 11.8; below it the cached loads are the faster ones: 3072 x 2048 (13 MB) 8.9 against 9.8.
constexpr size_t ONCE_BYTES = 24u << 20;

inline bool weights_once(const GemmArgs &a, int tiles_m) { return tiles_m == 1 && (size_t)a.N * a.K * 2 >= ONCE_BYTES; }

// The streaming kernel for a handful of rows (gemm_stream.hip): 16-column tiles per wave (1 or 2) where a layer whose K is
// cut into `split` parts should run on it, else 0
int gemm_stream_tiles(int M, int N, int K, int split, int glu);
hipError_t launch_gemm_stream(const GemmArgs &a, int tiles, int split, hipStream_t s);

// adds the partial tiles of a split layer and applies the epilogue (gemm.hip)
hipError_t launch_split_finish(const float *partial, const float *ssq_part, const Epilogue &e, int split,
                               const GemmArgs &a, hipStream_t s);
// the fused norm's row sums of squares by a launch of their own: ssq[split][M] in the workspace (gemm_panel.hip).
// Unsplit, only in a workspace that is the launch's own: the caller of a public operation may share one between streams.
// (A tile forced by the tuning call runs whatever it needs.)  -1: no norm
inline ptrdiff_t gemm_norm_bytes(const GemmArgs &a) { return !a.fused_norm ? -1 : a.ws && (a.own_ws || a.tile > 0) ? (ptrdiff_t)a.ws_bytes : 0; }
inline bool squares_fit(int M, size_t ws_bytes) { return (size_t)M * sizeof(float) <= GEMM_SSQ_BYTES && ws_bytes >= GEMM_SSQ_BYTES; }
hipError_t launch_row_squares(const GemmArgs &a, int split_k, int kt_per_split, float *ssq, hipStream_t s);
// the tile configurations (gemm_tiles_*.hip)
hipError_t dispatch_narrow(int tile, const GemmArgs &a, hipStream_t s, int split);  // 1-5
hipError_t dispatch_wide(int tile, const GemmArgs &a, hipStream_t s, int split);    // 6-10
hipError_t dispatch_tall(int tile, const GemmArgs &a, hipStream_t s, int split);    // 11-14
hipError_t prepare_tall();  // their function attributes, once per device
// the block kernel's (gemm_block.hip)
hipError_t dispatch_block(int tile, const GemmArgs &a, hipStream_t s, int split);  // 15-31
hipError_t prepare_block();
hipError_t dispatch_panel(int tile, const GemmArgs &a, hipStream_t s, int split);  // those of them on the panel kernel
hipError_t dispatch_panel_narrow(int tile, const GemmArgs &a, hipStream_t s, int split);
hipError_t prepare_panel();
hipError_t prepare_panel_narrow();
inline bool squares_before(int tile) { return (tile >= 15 && tile <= 17) || (tile >= 26 && tile <= 28); }  // a norm's row sums: a launch of their own
int block_groups(int tile);  // groups of waves that share a split K inside a workgroup (1: none)
bool block_takes(int tile, int M, int N, int K, int split, bool am, ptrdiff_t norm_ws);  // whether that tile can run such a layer

}  // namespace sf
