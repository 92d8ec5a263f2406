// fp32 linear layers  y[M][N] = x[M][K] . w[N][K]^T  of the small fp32 configuration, row-major weights.
//
// Such a layer is a few hundred KB of weights and a few dozen rows: nothing but latency.  A workgroup owns
// 16 * TM rows x 16 * TN columns and cuts K over its up to 16 waves; a wave loads its whole share of both
// operands in a few independent rounds of 16-byte loads straight into registers (no LDS, no barrier in the K
// loop) and multiplies with v_mfma_f32_16x16x4_f32 (full fp32 products and sums).  The waves' partial tiles meet
// in LDS once and are added in wave order, so a result depends on K alone, not on the rows batched with it.
// 20 x 256 x 1024: 143 us -> 5 us, 20 x 768 x 256: 39 us -> 5 us against a 64 x 64 tile with LDS staging, whose
// 4-16 workgroups walked K serially.
//
// On the way out: bias, residual, hooked copies of the block rows.  On the way in: RMSNorm (the gains multiply the
// rows as they arrive, the row factor the sums).  SwiGLU: the second column tile of a workgroup is the up
// projection of the first one's gate columns.
#include "sf_internal.h"

#include <algorithm>

namespace sf {
namespace {

constexpr int MAX_WAVES = 16;

__device__ __forceinline__ f32x4 keep(f32x4 v, bool yes) { return yes ? v : f32x4{0.f, 0.f, 0.f, 0.f}; }

// U: chunks of 16 positions a wave has in flight
template <int TM, int TN, int U>
__global__ __launch_bounds__(64 * MAX_WAVES) void linear_f32_kernel(
    const float *__restrict__ X, const float *__restrict__ W, const float *__restrict__ gain, float eps,
    const float *__restrict__ bias, const float *residual, float *Y, float *__restrict__ hooks, int hook_mask,
    int hook_q, int hook_qmax, int glu, int M, int N, int K, int chunks_per_wave) {
  extern __shared__ float part[];  // [waves][TM * TN][16][16] partial tiles, then [waves][16 * TM] sums of squares
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = blockDim.x >> 6;
  const int r = lane & 15, g = lane >> 4;
  const int m0 = blockIdx.y * 16 * TM;
  const int F = N >> 1;
  const int n0 = blockIdx.x * (glu ? 16 : 16 * TN);
  const int n_end = glu ? F : N;

  f32x4 acc[TM][TN];
  float ssq[TM];
#pragma unroll
  for (int a = 0; a < TM; ++a) {
    ssq[a] = 0.f;
#pragma unroll
    for (int b = 0; b < TN; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const float *xp[TM], *wp[TN];
#pragma unroll
  for (int a = 0; a < TM; ++a) xp[a] = X + (size_t)min(m0 + a * 16 + r, M - 1) * K;
#pragma unroll
  for (int b = 0; b < TN; ++b)  // with the gate, tile 1 holds the up rows of tile 0's gate rows
    wp[b] = W + (size_t)(min(n0 + (glu ? 0 : b * 16) + r, n_end - 1) + (glu ? b * F : 0)) * K;
  const int c0 = wave * chunks_per_wave, c1 = min(c0 + chunks_per_wave, (K + 15) / 16);
  const int whole = min(c1, K >> 4);  // the chunks before this one lie inside K
  auto product = [&](f32x4 (&x)[TM], const f32x4 (&w)[TN], const f32x4 &gains) __attribute__((always_inline)) {
    if (gain) {
#pragma unroll
      for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          ssq[a] += x[a][j] * x[a][j];
          x[a][j] *= gains[j];
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[a][j], w[b][j], acc[a][b], 0, 0, 0);
  };
  for (int c = c0; c < c1; c += U) {
    f32x4 xa[U][TM], wb[U][TN], gv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // lane (r, g) takes positions k .. k+3 of its row; product j of the four pairs element j of every lane
      const int kk = min((c + u) * 16 + g * 4, K - 4);
#pragma unroll
      for (int a = 0; a < TM; ++a) xa[u][a] = *reinterpret_cast<const f32x4 *>(xp[a] + kk);
#pragma unroll
      for (int b = 0; b < TN; ++b) wb[u][b] = *reinterpret_cast<const f32x4 *>(wp[b] + kk);
      gv[u] = gain ? *reinterpret_cast<const f32x4 *>(gain + kk) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    if (c + U > whole) {  // past the share or past K: zeros on all sides (a zero times an infinity is none)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool in = c + u < c1 && (c + u) * 16 + g * 4 < K;
#pragma unroll
        for (int a = 0; a < TM; ++a) xa[u][a] = keep(xa[u][a], in);
#pragma unroll
        for (int b = 0; b < TN; ++b) wb[u][b] = keep(wb[u][b], in);
        gv[u] = keep(gv[u], in);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) product(xa[u], wb[u], gv[u]);
  }

  constexpr int TILE = TM * TN * 256;
  float *sq = part + waves * TILE;
#pragma unroll
  for (int a = 0; a < TM; ++a) {
#pragma unroll
    for (int b = 0; b < TN; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) part[wave * TILE + (a * TN + b) * 256 + (g * 4 + v) * 16 + r] = acc[a][b][v];
    if (gain) {
      float t = ssq[a];
      t += __shfl_xor(t, 16);
      t += __shfl_xor(t, 32);
      if (g == 0) sq[wave * 16 * TM + a * 16 + r] = t;
    }
  }
  __syncthreads();
  const int outs = glu ? TM * 256 : TILE;
  for (int x = tid; x < outs; x += blockDim.x) {
    const int a = glu ? x / 256 : x / (TN * 256), b = glu ? 0 : x / 256 % TN, row = x / 16 % 16, c = x % 16;
    const int m = m0 + a * 16 + row, n = n0 + b * 16 + c;
    if (m >= M || n >= n_end) continue;
    auto total = [&](int tile) {
      float s = 0.f;
      for (int w = 0; w < waves; ++w) s += part[w * TILE + (a * TN + tile) * 256 + row * 16 + c];
      return s;
    };
    float rinv = 1.f;
    if (gain) {
      float t = 0.f;
      for (int w = 0; w < waves; ++w) t += sq[w * 16 * TM + a * 16 + row];
      rinv = 1.0f / sqrtf(t / (float)K + eps);
    }
    float v = total(b) * rinv;
    if (TN > 1 && glu) {
      const float up = total(TN - 1) * rinv;
      Y[(size_t)m * F + n] = v / (1.0f + expf(-v)) * up;
      continue;
    }
    if (bias) v += bias[n];
    if (residual) v += residual[(size_t)m * N + n];
    Y[(size_t)m * N + n] = v;
    if (hooks) {
      const size_t hrow = ((size_t)(m / hook_q) * hook_qmax + m % hook_q) * 4;
#pragma unroll
      for (int h = 1; h < 4; ++h)
        if (hook_mask >> h & 1) hooks[(hrow + h) * N + n] = v;
    }
  }
}

template <int TM, int TN>
hipError_t run(const GemmArgs &a, hipStream_t s) {
  const int chunks = (a.K + 15) / 16;
  // two chunks or more per wave: K = 256 takes 8 waves, K = 512 and above 16 (8 with the gate, whose partial
  // tiles would outgrow 64 KiB); never a matter of M
  const int most = a.glu ? MAX_WAVES / 2 : MAX_WAVES;
  int waves = 1;
  while (waves < most && waves * 4 <= chunks) waves *= 2;
  const int per_wave = (chunks + waves - 1) / waves;
  const int cols = a.glu ? a.N / 2 : a.N, bn = a.glu ? 16 : 16 * TN;
  const dim3 grid((cols + bn - 1) / bn, (a.M + 16 * TM - 1) / (16 * TM));
  const size_t lds = (size_t)waves * (TM * TN * 256 + 16 * TM) * sizeof(float);
  auto launch = [&](auto kernel) {
    kernel<<<grid, 64 * waves, lds, s>>>(
        (const float *)a.x, (const float *)a.w, (const float *)a.gain_f32, a.norm_eps, (const float *)a.bias,
        (const float *)a.residual, (float *)a.y, (float *)a.hooks, a.hook_mask, a.hook_q, a.hook_qmax, a.glu, a.M, a.N,
        a.K, per_wave);
  };
  if (per_wave <= 2) launch(&linear_f32_kernel<TM, TN, 2>); else launch(&linear_f32_kernel<TM, TN, 4>);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_f32(const GemmArgs &a, hipStream_t s) {
  if (a.glu) return a.M <= 16 ? run<1, 2>(a, s) : run<2, 2>(a, s);
  return a.M <= 16 ? run<1, 1>(a, s) : run<2, 1>(a, s);
}

}  // namespace sf
