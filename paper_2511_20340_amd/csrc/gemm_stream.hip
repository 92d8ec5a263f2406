// bf16 linear layers of at most 32 rows: the batch is a handful of sequences, the weights are all there is to
// move, and what counts is how soon every compute unit has its share of them in flight.
//
// A workgroup owns 16 or 32 weight rows (output columns) over the WHOLE of K; its eight waves cut K among themselves,
// stream their packed weight fragments and the few activation rows straight into registers (no LDS, no barrier in the
// loop) and multiply with v_mfma_f32_16x16x32_bf16.  The eight partial tiles meet in LDS and are added in wave order,
// then the epilogue runs on rows of 8 columns.  So no K split over workgroups and no second launch is needed to fill
// the chip, and the order of a sum depends on K alone.
// 5 rows, against the tiled kernel with its K split over workgroups: 2048 x 2048 7.9 -> 4.8 us, 3072 x 2048 9.1 -> 5.4,
// 4096 x 4096 12.2 -> 9.3, 6144 x 4096 15.3 -> 11.7.
#include "gemm_common.h"

namespace sf {
namespace {

constexpr int SWAVES = 8;

// TM: 16-row tiles of activations, TN: 16-column tiles of weights; NORM: the rows are to be RMS-normalised (the gains
// are folded into the weights, the row factor is formed here); ONCE: non-temporal weight loads
template <int TM, int TN, int NORM, int ONCE>
__global__ __launch_bounds__(64 * SWAVES, 4) void gemm_stream_kernel(const bf16_t *__restrict__ A,
                                                                     const uint4 *__restrict__ Wp, const Epilogue e,
                                                                     int M, int N, int K, float eps) {
  constexpr int U = 8 / (TM + TN);  // 32-position chunks per batch; two batches are in flight
  constexpr int TILE = TM * TN * 256;
  __shared__ __attribute__((aligned(16))) float part[SWAVES * TILE];
  __shared__ float sq[SWAVES][16 * TM];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 15, kg = lane >> 4;
  const int k_steps = (K + 15) >> 4, chunks = (K + 31) >> 5;
  const int per_wave = (chunks + SWAVES - 1) / SWAVES;
  const int c0 = wave * per_wave, c1 = min(c0 + per_wave, chunks);
  const int n0 = blockIdx.x * 16 * TN;

  const bf16_t *ap[TM];
#pragma unroll
  for (int a = 0; a < TM; ++a) ap[a] = A + (size_t)min(a * 16 + r, M - 1) * K;
  // column tile b: rows (n0 + 16 b) % 32 .. +15 of packed row block (n0 + 16 b) / 32; a lane's 8 positions sit in unit
  // 2 c + kg / 2 of chunk c, half kg % 2
  const uint4 *wp[TN];
#pragma unroll
  for (int b = 0; b < TN; ++b) {
    const int n = n0 + b * 16;
    wp[b] = Wp + (size_t)(n >> 5) * k_steps * 64 + (kg & 1) * 32 + (n & 16) + r;
  }

  f32x4 acc[TM][TN];
  float ssq[TM];
#pragma unroll
  for (int a = 0; a < TM; ++a) {
    ssq[a] = 0.f;
#pragma unroll
    for (int b = 0; b < TN; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  uint4 wf[2][U][TN], af[2][U][TM];
  auto load = [&](int buf, int c) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int unit = min(2 * (c + u) + (kg >> 1), k_steps - 1);
#pragma unroll
      for (int b = 0; b < TN; ++b) wf[buf][u][b] = load_unit<ONCE>(wp[b] + (size_t)unit * 64);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int a = 0; a < TM; ++a)
        af[buf][u][a] = *reinterpret_cast<const uint4 *>(ap[a] + min((c + u) * 32 + kg * 8, K - 8));
  };
  auto multiply = [&](int buf, int c) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool live = c + u < c1 && (c + u) * 32 + kg * 8 < K;  // past the share or past K: zeros
#pragma unroll
      for (int a = 0; a < TM; ++a) {
        uint4 v = af[buf][u][a];
        v.x = live ? v.x : 0u; v.y = live ? v.y : 0u; v.z = live ? v.z : 0u; v.w = live ? v.w : 0u;
        if (NORM) {
          float t = ssq[a];
          t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, v.x), __builtin_bit_cast(bf16x2, v.x), t, false);
          t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, v.y), __builtin_bit_cast(bf16x2, v.y), t, false);
          t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, v.z), __builtin_bit_cast(bf16x2, v.z), t, false);
          t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, v.w), __builtin_bit_cast(bf16x2, v.w), t, false);
          ssq[a] = t;
        }
#pragma unroll
        for (int b = 0; b < TN; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, v),
                                                              __builtin_bit_cast(bf16x8, wf[buf][u][b]), acc[a][b], 0, 0, 0);
      }
    }
  };
  if (c0 < c1) {
    load(0, c0);
    for (int c = c0; c < c1; c += 2 * U) {
      load(1, c + U);
      __builtin_amdgcn_sched_barrier(0);  // a batch is requested whole before the one ahead of it is multiplied
      multiply(0, c);
      load(0, c + 2 * U);
      __builtin_amdgcn_sched_barrier(0);
      multiply(1, c + U);
    }
  }

#pragma unroll
  for (int a = 0; a < TM; ++a) {
#pragma unroll
    for (int b = 0; b < TN; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) part[wave * TILE + (a * TN + b) * 256 + (kg * 4 + v) * 16 + r] = acc[a][b][v];
    if (NORM) {
      float t = ssq[a];
      t += __shfl_xor(t, 16);
      t += __shfl_xor(t, 32);
      if (kg == 0) sq[wave][a * 16 + r] = t;
    }
  }
  __syncthreads();
  // one thread per row and 8 columns (with the gate: 8 features, columns f and f + 16 of the pair of tiles)
  const int groups = e.glu ? TN : 2 * TN;
  if (tid >= 16 * TM * groups) return;
  const int row = tid / groups, g = tid % groups, a = row >> 4;
  const int c8 = e.glu ? (g >> 1) * 32 + (g & 1) * 8 : g * 8;
  if (row >= M) return;
  auto total = [&](int col, float (&v)[8]) {
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = 0.f;
#pragma unroll
    for (int w = 0; w < SWAVES; ++w) {
      const float *p = part + w * TILE + (a * TN + (col >> 4)) * 256 + (row & 15) * 16 + (col & 15);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const f32x4 q = *reinterpret_cast<const f32x4 *>(p + j * 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) v[j * 4 + i] += q[i];
      }
    }
  };
  float rinv = 1.f;
  if (NORM) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < SWAVES; ++w) t += sq[w][row];
    rinv = 1.0f / sqrtf(t / (float)K + eps);
  }
  float v[8];
  total(c8, v);
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] *= rinv;
  if (e.glu) {
    const int f = (n0 >> 1) + g * 8;
    float up[8];
    total((c8 + 16) & (16 * TN - 1), up);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = v[i] / (1.0f + __expf(-v[i])) * (up[i] * rinv);
    if (f < (N >> 1)) store8(reinterpret_cast<bf16_t *>(e.y) + (size_t)row * (N >> 1) + f, v, e.vec);
    return;
  }
  const int col = n0 + c8;
  if (col < N) finish_row8(e, row, col, N, v);
}

template <int TM, int TN, int NORM>
hipError_t run(const GemmArgs &a, hipStream_t s) {
  const Epilogue e = make_epilogue(a);
  const dim3 grid((a.N + 16 * TN - 1) / (16 * TN));
  if (weights_once(a, 1))
    gemm_stream_kernel<TM, TN, NORM, 1><<<grid, 64 * SWAVES, 0, s>>>((const bf16_t *)a.x, (const uint4 *)a.w, e, a.M, a.N,
                                                                     a.K, a.norm_eps);
  else
    gemm_stream_kernel<TM, TN, NORM, 0><<<grid, 64 * SWAVES, 0, s>>>((const bf16_t *)a.x, (const uint4 *)a.w, e, a.M, a.N,
                                                                     a.K, a.norm_eps);
  return hipGetLastError();
}
template <int TM, int TN>
hipError_t run(const GemmArgs &a, hipStream_t s) {
  return a.fused_norm ? run<TM, TN, 1>(a, s) : run<TM, TN, 0>(a, s);
}

}  // namespace

// Where the streaming kernel is the faster one (5 / 16 / 30 rows, weights cold, against the tiled kernel):
// * every compute unit gets one workgroup, or two: 16 columns each up to 256 workgroups, then 32.  5120 x 5120 at 5
//   rows: 12.2 us as 160 workgroups of 32 columns, 17.4 as 320 of 16, tiled 14.4; 16384 x 2048 as 512: 15.5, tiled 18.4;
//   28672 x 4096 as 896: 44.3, tiled 40.3.
// * the rows are read by every workgroup, so they have to stay few beside 16 or 32 weight rows: at 16 rows 6144 x 4096
//   13.0 against 15.7 and 5120 x 5120 14.9 against 15.1, but 4096 x 14336 25.9 against 25.0 (at 5 rows 21.0 against 24.3);
//   at 30 rows 3072 x 2048 8.2 against 10.4 and 4096 x 4096 12.8 against 13.8, but 7168 x 5120 20.2 against 19.3.
// The choice goes by the rows a layer is planned for, not by those of one call: a row's sums have one order.
int gemm_stream_columns(int plan_M, int N, int K, int glu) {
  const bool rows_ok = plan_M <= 8 || (plan_M <= 16 && K <= 6144) || (plan_M <= 32 && (size_t)N * K <= (17u << 20));
  if (!rows_ok) return 0;
  if (!glu && N <= 256 * 16) return 16;
  const int wgs = (N + 31) / 32;
  return wgs <= 256 || (wgs > 448 && wgs <= 512) ? 32 : 0;
}

hipError_t launch_gemm_stream(const GemmArgs &a, int columns, hipStream_t s) {
  if (a.M <= 16) return columns == 32 ? run<1, 2>(a, s) : run<1, 1>(a, s);
  return columns == 32 ? run<2, 2>(a, s) : run<2, 1>(a, s);
}

}  // namespace sf
