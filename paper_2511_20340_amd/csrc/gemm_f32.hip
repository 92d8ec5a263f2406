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

// Many rows: the same sums without LDS.  A workgroup of 2 x 2 waves owns 128 rows x 64 columns (with the gate 64 gate and
// up rows of the weight); a wave takes 64 x 32 of them over the whole of K, one share after the other in wave order of the
// kernel above, and adds a share's products to the total when the share ends: the same bits.  A fragment loaded from
// memory is used four or two times here and once or twice there.  8192 x 2048 x 256 174 -> 111 us, 2048 x 4096 x 1024
// 415 -> 194, 8192 x 4096 x 4096 5760 -> 2794.
constexpr int RM = 4, RN = 2;  // 16-row and 16-column tiles of a wave
constexpr int ROWS_BM = 2 * RM * 16, ROWS_BN = 2 * RN * 16;

__global__ __launch_bounds__(256) void linear_f32_rows_kernel(
    const float *__restrict__ X, const float *__restrict__ W, const float *__restrict__ gain, float eps,
    const float *__restrict__ bias, const float *residual, float *Y, float *__restrict__ hooks, int hook_mask,
    int hook_q, int hook_qmax, int glu, int M, int N, int K, int chunks_per_wave) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, g = lane >> 4;
  const int m0 = blockIdx.y * ROWS_BM + (wave >> 1) * RM * 16;
  const int F = N >> 1, n_end = glu ? F : N;
  const int n0 = (blockIdx.x * 2 + (wave & 1)) * (glu ? 16 : RN * 16);
  const int chunks = (K + 15) / 16;
  const float *xp[RM], *wp[RN];
#pragma unroll
  for (int a = 0; a < RM; ++a) xp[a] = X + (size_t)min(m0 + a * 16 + r, M - 1) * K;
#pragma unroll
  for (int b = 0; b < RN; ++b) wp[b] = W + (size_t)(min(n0 + (glu ? 0 : b * 16) + r, n_end - 1) + (glu ? b * F : 0)) * K;

  f32x4 acc[RM][RN], sum[RM][RN];
  float ssq[RM], sq[RM];
#pragma unroll
  for (int a = 0; a < RM; ++a) {
    ssq[a] = sq[a] = 0.f;
#pragma unroll
    for (int b = 0; b < RN; ++b) acc[a][b] = sum[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  f32x4 xa[2][RM], wb[2][RN], gv[2];
  auto load = [&](int buf, int c) __attribute__((always_inline)) {
    const int kk = min(c * 16 + g * 4, K - 4);
#pragma unroll
    for (int a = 0; a < RM; ++a) xa[buf][a] = *reinterpret_cast<const f32x4 *>(xp[a] + kk);
#pragma unroll
    for (int b = 0; b < RN; ++b) wb[buf][b] = *reinterpret_cast<const f32x4 *>(wp[b] + kk);
    gv[buf] = gain ? *reinterpret_cast<const f32x4 *>(gain + kk) : f32x4{0.f, 0.f, 0.f, 0.f};
  };
  int left = chunks_per_wave;  // chunks of the current share
  auto multiply = [&](int buf, int c) __attribute__((always_inline)) {
    if (c * 16 + 16 > K) {
      const bool in = c * 16 + g * 4 < K;
#pragma unroll
      for (int a = 0; a < RM; ++a) xa[buf][a] = keep(xa[buf][a], in);
#pragma unroll
      for (int b = 0; b < RN; ++b) wb[buf][b] = keep(wb[buf][b], in);
      gv[buf] = keep(gv[buf], in);
    }
    if (gain) {
#pragma unroll
      for (int a = 0; a < RM; ++a)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          ssq[a] += xa[buf][a][j] * xa[buf][a][j];
          xa[buf][a][j] *= gv[buf][j];
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int a = 0; a < RM; ++a)
#pragma unroll
        for (int b = 0; b < RN; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[buf][a][j], wb[buf][b][j], acc[a][b], 0, 0, 0);
    if (--left == 0 || c == chunks - 1) {
      left = chunks_per_wave;
#pragma unroll
      for (int a = 0; a < RM; ++a) {
#pragma unroll
        for (int b = 0; b < RN; ++b) {
          sum[a][b] += acc[a][b];
          acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        if (gain) {
          float t = ssq[a];
          t += __shfl_xor(t, 16);
          t += __shfl_xor(t, 32);
          sq[a] += t;
          ssq[a] = 0.f;
        }
      }
    }
  };
  load(0, 0);
  for (int c = 0; c < chunks; c += 2) {
    load(1, min(c + 1, chunks - 1));
    multiply(0, c);
    if (c + 1 == chunks) break;
    load(0, min(c + 2, chunks - 1));
    multiply(1, c + 1);
  }

#pragma unroll
  for (int a = 0; a < RM; ++a) {
    const float rinv = gain ? 1.0f / sqrtf(sq[a] / (float)K + eps) : 1.f;  // of row a * 16 + r
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float f = __shfl(rinv, g * 4 + v);
      const int m = m0 + a * 16 + g * 4 + v;
      if (glu) {
        const int n = n0 + r;
        const float x = sum[a][0][v] * f, up = sum[a][1][v] * f;
        if (m < M && n < F) Y[(size_t)m * F + n] = x / (1.0f + expf(-x)) * up;
        continue;
      }
#pragma unroll
      for (int b = 0; b < RN; ++b) {
        const int n = n0 + b * 16 + r;
        if (m >= M || n >= N) continue;
        float x = sum[a][b][v] * f;
        if (bias) x += bias[n];
        if (residual) x += residual[(size_t)m * N + n];
        Y[(size_t)m * N + n] = x;
        if (hooks) {
          const size_t hrow = ((size_t)(m / hook_q) * hook_qmax + m % hook_q) * 4;
#pragma unroll
          for (int h = 1; h < 4; ++h)
            if (hook_mask >> h & 1) hooks[(hrow + h) * N + n] = x;
        }
      }
    }
  }
}

// K's shares: two chunks or more each; K = 256 has 8, K = 512 and above 16 (8 with the gate, whose partial tiles would
// outgrow 64 KiB); never a matter of M
int shares_of(const GemmArgs &a) {
  const int chunks = (a.K + 15) / 16, most = a.glu ? MAX_WAVES / 2 : MAX_WAVES;
  int waves = 1;
  while (waves < most && waves * 4 <= chunks) waves *= 2;
  return waves;
}

template <int TM, int TN>
hipError_t run(const GemmArgs &a, hipStream_t s) {
  const int chunks = (a.K + 15) / 16;
  const int waves = shares_of(a);
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
  // From about ten workgroups of the small kernel per compute unit on, the chip is full either way and the larger tile is
  // the faster one, unless rows fill little of it: 512 x 4096 x 1024 (4096 workgroups) 106 -> 56 us, 768 x 2048 x 256 (3072)
  // 20.2 -> 19.2, but 512 x 2048 x 512 (2048) 26 against 31 and 33 x 32000 x 1024 86 against 93.
  if (a.M >= 64 && (long)((a.N + 15) / 16) * ((a.M + 31) / 32) >= 2560) {
    const int shares = shares_of(a), chunks = (a.K + 15) / 16;
    const int cols = a.glu ? a.N / 2 : a.N, bn = a.glu ? ROWS_BN / 2 : ROWS_BN;
    linear_f32_rows_kernel<<<dim3((cols + bn - 1) / bn, (a.M + ROWS_BM - 1) / ROWS_BM), 256, 0, s>>>(
        (const float *)a.x, (const float *)a.w, (const float *)a.gain_f32, a.norm_eps, (const float *)a.bias,
        (const float *)a.residual, (float *)a.y, (float *)a.hooks, a.hook_mask, a.hook_q, a.hook_qmax, a.glu, a.M, a.N,
        a.K, (chunks + shares - 1) / shares);
    return hipGetLastError();
  }
  if (a.glu) return a.M <= 16 ? run<1, 2>(a, s) : run<2, 2>(a, s);
  return a.M <= 16 ? run<1, 1>(a, s) : run<2, 1>(a, s);
}

}  // namespace sf
